// GEMMs of the layer: C = epilogue(A W^T), A [M, K] row-major, W [N, K]
// (the nn.Linear orientation) stored in 64x64 tiles: tile (i, j) covers rows
// 64i.. and columns 64j.., sits at tile index i * ceil(K/64) + j, and is
// row-major inside (64 rows of 64 elements). Every 64-row by 64-k slab a
// workgroup streams is then one contiguous 8 KiB (bf16) block of HBM rather
// than 64 strided 128-byte pieces. fp32 accumulation (gfx950).
//
//  * gemm_tile_kernel (gemm_tile.h): M > 64, 256x256 down to 64x64 workgroup
//    tiles chosen by gemm_tile_plan.
//  * gemm_skinny_kernel: decode-sized M (<= 64). Streams W once from HBM
//    with 16-byte loads, one 16-column MFMA block per wave, activations
//    staged in LDS and shared by the workgroup's four waves; K may be split
//    across workgroups, fp32 partials then reduced in split order by
//    gemm_reduce_kernel. HBM-bound (AI = M FLOP/byte).
//  * gemm_f32_kernel: fp32 layers, fp32 MFMA straight from global memory.
//
// Epilogues: store, residual add (C = R + A W^T) and SwiGLU (W rows
// interleaved gate/up in blocks of 32; C[:, j] = silu(gate_j) * up_j).
#include "gemm_tile.h"

#include <mutex>

namespace ps {

// ==================================================================== skinny
// Decode-sized M (<= 64): the weight stream is the whole cost (AI = M
// FLOP/byte). A workgroup owns 64 WN weight rows (output columns, WN 1, 2 or 4) and a K
// range; its four waves own 16 WN rows each. Stages of 64 k hold the
// activation tile [16 MB rows][64] and the weight tile [64 WN rows][64];
// both are filled by global->LDS DMA into an NS-deep ring, so the bytes in
// flight cost no registers, and one barrier per stage recycles the slot.
// LDS rows are 128 B with 16-byte chunks XOR-swizzled by row % 8 (the DMA
// lane order is chosen so the fill lands swizzled). Per 32-wide k step a
// wave does MB x WN v_mfma_f32_16x16x32_bf16 with A = activations, B = W.
// With one K split the epilogue is applied from registers; otherwise fp32
// partials go to the workspace and gemm_reduce_kernel sums them in split
// order.
namespace skinny {
constexpr int NT = 256;
constexpr int KS = 64;    // k per stage
constexpr int MAXM = 64;
template <int WN>
constexpr int ring() { return WN == 4 ? 3 : 4; }  // stages; three of the widest are as many bytes in flight as six of 128 rows
template <int MB, int WN>
constexpr size_t lds_bytes() { return (size_t)ring<WN>() * (16 * MB + 64 * WN) * KS * 2; }
}  // namespace skinny

template <int MB, int WN, int EPI, typename TR, typename TC, bool DIRECT>
__global__ __launch_bounds__(256) void gemm_skinny_kernel(const bf16_t* __restrict__ A, const bf16_t* __restrict__ W,
                                                          float* __restrict__ part, const TR* __restrict__ R,
                                                          TC* __restrict__ C, int M, int N, int K, int S) {
  using namespace skinny;
  static_assert(!(DIRECT && EPI == 2) || WN >= 2, "in-kernel SwiGLU pairs gate and up blocks per wave");
  constexpr int NS = ring<WN>();
  static_assert(KS == kWTile, "one W tile per stage");
  constexpr int AROWS = 16 * MB, WROWS = 64 * WN;
  constexpr int STAGE = (AROWS + WROWS) * KS;  // bf16 elements
  constexpr int TA = AROWS / 8;                // A DMA instructions per stage (8 rows each), round-robin
  constexpr int WI = WROWS / 8 / 4;            // W DMA instructions per wave per stage
  extern __shared__ __attribute__((aligned(16))) bf16_t smem[];
  const int n0 = blockIdx.x * WROWS;
  const int split = blockIdx.y;
  // split `split` of S takes 64-k stages [split TT / S, (split + 1) TT / S): near-equal ranges for any S
  const int TT = K / KS;
  const int st0 = split * TT / S;
  const int T = (split + 1) * TT / S - st0;
  const int kb = st0 * KS;
  const int kps = T * KS;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  const int g = lane >> 4, c = lane & 15;
  // DMA lane mapping: an instruction fills 8 rows; lane l lands in row l/8 at
  // chunk l%8, which holds global chunk (l%8) ^ (row%8)
  const int drow = lane >> 3, dch = (lane & 7) ^ (lane >> 3);
  const int n_ai = (TA - wave + 3) / 4;  // this wave's A instructions (0..2)
  // DMA sources: buffer resources at the split's first activation column and
  // at the workgroup's first W tile of the split, 32-bit lane byte offsets
  const __amdgpu_buffer_rsrc_t rA = buffer_rsrc(A + kb, (uint32_t)((long)(M - 1) * K + kps) * 2);
  const __amdgpu_buffer_rsrc_t rW = buffer_rsrc(W + ((long)(n0 >> 6) * (K / 64) + kb / 64) * kWTileElts,
                                                (uint32_t)((WN - 1) * (K / 64) + kps / 64) * kWTileElts * 2);
  uint32_t aoff[2], woff[WI];
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int row = (wave + 4 * i) * 8 + drow;
    aoff[i] = ((uint32_t)min(row, M - 1) * K + dch * 8) * 2;
  }
  // tiled W: the stage's 64 k of each 64-row block is one contiguous tile
#pragma unroll
  for (int i = 0; i < WI; ++i) {
    const int r = (wave * WI + i) * 8 + drow;  // row within the workgroup's WN blocks
    woff[i] = ((uint32_t)(r >> 6) * (K / 64) * kWTileElts + (r & 63) * 64 + dch * 8) * 2;
  }
  auto dma = [&](int t, int slot) {
    bf16_t* st = smem + slot * STAGE;
#pragma unroll
    for (int i = 0; i < 2; ++i)
      if (i < n_ai) load_lds16_buf(rA, aoff[i] + t * KS * 2, st + (wave + 4 * i) * 8 * KS);
#pragma unroll
    for (int i = 0; i < WI; ++i) load_lds16_buf_nt(rW, woff[i] + t * kWTileElts * 2, st + AROWS * KS + (wave * WI + i) * 8 * KS);
  };
  // this wave's own fills older than the most recent stage have landed
  auto wait_prev_stage = [&]() {
    if (n_ai == 2) wait_vmcnt_lgkm0<(NS - 2) * (WI + 2)>();
    else if (n_ai == 1) wait_vmcnt_lgkm0<(NS - 2) * (WI + 1)>();
    else wait_vmcnt_lgkm0<(NS - 2) * WI>();
  };
  auto swz = [](int row, int ch) { return row * KS + ((ch ^ (row & 7)) << 3); };
  // weight rows of n-block nb for this wave; for SwiGLU with WN 2 block 0 is a
  // gate block and block 1 the matching up block of the 32-row interleave, with
  // WN 4 a wave's blocks 0, 1 are gate and 2, 3 up as they lie
  auto wrow = [&](int nb) {
    if constexpr (EPI == 2 && WN == 2) {
      const int q = wave >> 1, h = wave & 1;
      return 64 * q + 32 * nb + 16 * h + c;
    } else {
      return wave * 16 * WN + nb * 16 + c;
    }
  };
  f32x4_t acc[WN][MB];
#pragma unroll
  for (int nb = 0; nb < WN; ++nb)
#pragma unroll
    for (int i = 0; i < MB; ++i) acc[nb][i] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  auto compute = [&](int slot) {
    const bf16_t* st = smem + slot * STAGE;
    const bf16_t* wt = st + AROWS * KS;
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      bf16x8_t wf[WN];
#pragma unroll
      for (int nb = 0; nb < WN; ++nb) wf[nb] = __builtin_bit_cast(bf16x8_t, *(const uint4*)(wt + swz(wrow(nb), 4 * j + g)));
#pragma unroll
      for (int i = 0; i < MB; ++i) {
        const bf16x8_t af = __builtin_bit_cast(bf16x8_t, *(const uint4*)(st + swz(16 * i + c, 4 * j + g)));
#pragma unroll
        for (int nb = 0; nb < WN; ++nb)
          acc[nb][i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(af, wf[nb], acc[nb][i], 0, 0, 0);
      }
    }
  };
#pragma unroll
  for (int d = 0; d < NS - 1; ++d)
    if (d < T) dma(d, d);
  int slot = 0, fill = NS - 1, t = 0;
  // steady state: every stage refills the slot freed by the previous one
  for (; t + NS - 1 < T; ++t) {
    wait_prev_stage();
    lds_barrier();
    dma(t + NS - 1, fill);
    compute(slot);
    if (++slot == NS) slot = 0;
    if (++fill == NS) fill = 0;
  }
  for (; t < T; ++t) {  // drain
    wait_vmcnt_lgkm0<0>();
    lds_barrier();
    compute(slot);
    if (++slot == NS) slot = 0;
  }
  // acc[nb][i][r] = C[16i + 4g + r][n0 + wrow(nb)]
  if constexpr (DIRECT) {
#pragma unroll
    for (int i = 0; i < MB; ++i)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int row = 16 * i + 4 * g + r;
        if (row >= M) continue;
        if constexpr (EPI == 2) {
#pragma unroll
          for (int nb = 0; nb < WN / 2; ++nb) {
            const int col = n0 / 2 + (WN == 4 ? 32 * wave + 16 * nb : 16 * wave) + c;
            st_elt<TC>(C, (long)row * (N / 2) + col, silu_fast(acc[nb][i][r]) * acc[nb + WN / 2][i][r]);
          }
        } else {
#pragma unroll
          for (int nb = 0; nb < WN; ++nb) {
            const long idx = (long)row * N + n0 + wrow(nb);
            float v = acc[nb][i][r];
            if constexpr (EPI == 1) v += ld_elt<TR>(R, idx);
            st_elt<TC>(C, idx, v);
          }
        }
      }
  } else {
    float* pp = part + (long)split * M * N;
#pragma unroll
    for (int nb = 0; nb < WN; ++nb)
#pragma unroll
      for (int i = 0; i < MB; ++i)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int row = 16 * i + 4 * g + r;
          if (row < M) pp[(long)row * N + n0 + wrow(nb)] = acc[nb][i][r];
        }
  }
}

// Sum split partials in split order, then apply the epilogue.
template <int EPI, typename TR, typename TC>
__global__ __launch_bounds__(256) void gemm_reduce_kernel(const float* __restrict__ part, const TR* __restrict__ R,
                                                          TC* __restrict__ C, int M, int N, int S) {
  const long total = (EPI == 2) ? (long)M * (N / 2) : (long)M * N;
  for (long e = (long)blockIdx.x * 256 + threadIdx.x; e < total; e += (long)gridDim.x * 256) {
    if constexpr (EPI == 2) {
      const int ldc = N / 2;
      const long row = e / ldc;
      const int j = (int)(e - row * ldc);
      const int gcol = (j / kGateUpBlock) * (2 * kGateUpBlock) + (j % kGateUpBlock);
      float gs = 0.f, us = 0.f;
      for (int s = 0; s < S; ++s) {
        gs += part[((long)s * M + row) * N + gcol];
        us += part[((long)s * M + row) * N + gcol + kGateUpBlock];
      }
      st_elt<TC>(C, e, silu_fast(gs) * us);
    } else {
      float v = 0.f;
      for (int s = 0; s < S; ++s) v += part[(long)s * M * N + e];
      if constexpr (EPI == 1) v += ld_elt<TR>(R, e);
      st_elt<TC>(C, e, v);
    }
  }
}

// ======================================================================= f32
// fp32 layers on v_mfma_f32_16x16x4_f32 (fp32 products and sums; twice the
// vector rate without packed instructions). A wave holds RB x CB blocks of 16
// rows x 16 columns and reads its operands straight from global memory: in a
// 16-k step lane (h, r) loads k 4h .. 4h+3 of row r as one 16-byte access, and
// MFMA j takes element j of every lane, i.e. k j, 4+j, 8+j, 12+j - the same
// four for A and W, so any such order is a correct product. The step's rows
// are 64-byte segments; the next 64-k tile's loads are issued before this
// tile's MFMAs.
//
// These launches are short (the tiny layer: 0.1 to 4 MFLOP per wave), so what
// bounds them is the chain load - multiply - store and the number of
// workgroups in flight, not arithmetic. Two arrangements of a workgroup's four
// waves:
//  * KSPLIT: all four on the same 16 RB x 16 CB outputs, each over a quarter
//    of K's 64-wide tiles; partial sums meet in LDS and are added in wave
//    order. Many small tiles, a quarter of the chain each.
//  * else: 2 x 2 waves on 32 RB x 32 CB outputs, the whole K each: operands
//    are read once per 64 x 64 outputs, for launches that fill the chip.
// Measured (us, one launch): 4 x 512 x 256 (M, N, K) 33 -> 7.5 and
// 4 x 256 x 1024 124 -> 7.7 (both now a launch's own cost), 100 x 4096 x 4096
// 650 -> 73, 4096^3 2824 -> 1088 (126 TFLOP/s; torch 145), against 64 x 64
// LDS tiles on the vector ALU; the error against 64 bits is the same or half.
// SwiGLU: a wave's column block c comes with the matching up block (32 rows
// of W further on), so gate and up of one output sit in one lane.
// VEC: A rows can be read 16 bytes at a time (K a multiple of 4).
// NORM: A is the RMSNorm of the rows given, x / sqrt(mean x^2 + eps) * g. The
// gain goes onto the operands, the rows' sums of squares come from the same
// registers, and the root scales the finished sums, so the norm costs no load
// and no wait of its own; its launch (2.5 us on the stream and 2.3 on the host)
// goes. The leading workgroups then carry a call's metadata upload.
namespace f32g {
constexpr int NT = 256;
}
template <int RB, int CB, bool KSPLIT, bool VEC, bool NORM, int EPI, typename TR, typename TC>
__global__ __launch_bounds__(256) void gemm_f32_kernel(const float* __restrict__ A, const float* __restrict__ W,
                                                       const TR* __restrict__ R, TC* __restrict__ C, int M, int N,
                                                       int K, const float* __restrict__ gain, float eps, UploadJob up) {
  static_assert(!NORM || (KSPLIT && VEC), "the fused norm is for the small arrangements");
  int bx = blockIdx.x;
  if constexpr (NORM) {
    bx -= up.blocks;
    if (bx < 0) {
      if (blockIdx.y == 0) upload_block(up, blockIdx.x);
      return;
    }
  }
  constexpr int WB = EPI == 2 ? 2 * CB : CB;  // W blocks per wave
  constexpr int MW = KSPLIT ? 1 : 2;          // waves along each side of the workgroup tile
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int h = lane >> 4, r16 = lane & 15;
  const int m0 = (blockIdx.y * MW + (KSPLIT ? 0 : wave >> 1)) * 16 * RB;
  const int c0 = (bx * MW + (KSPLIT ? 0 : wave & 1)) * 16 * CB;  // output column
  const int kt = (K + kWTile - 1) / kWTile;
  const int t0 = KSPLIT ? wave * kt / 4 : 0, t1 = KSPLIT ? (wave + 1) * kt / 4 : kt;
  // W row of block b at this lane's r16 (rows past N read row 0 of the tile
  // grid's last block, results unused)
  const int n_pad = (N + kWTile - 1) / kWTile * kWTile;
  const float* wp[WB];
#pragma unroll
  for (int b = 0; b < WB; ++b) {
    int n;
    if constexpr (EPI == 2) {
      const int c = c0 + (b >> 1) * 16;  // output columns 32 i .. come from W rows 64 i .. (gate) and 64 i + 32 .. (up)
      n = c / kGateUpBlock * (2 * kGateUpBlock) + c % kGateUpBlock + (b & 1) * kGateUpBlock + r16;
    } else {
      n = c0 + b * 16 + r16;
    }
    n = min(n, n_pad - 1);
    wp[b] = W + ((long)(n / kWTile) * kt) * kWTileElts + (n % kWTile) * kWTile + 4 * h;
  }
  const float* ap[RB];
#pragma unroll
  for (int i = 0; i < RB; ++i) ap[i] = A + (long)min(m0 + 16 * i + r16, M - 1) * K + 4 * h;
  f32x4_t acc[RB][WB];
#pragma unroll
  for (int i = 0; i < RB; ++i)
#pragma unroll
    for (int b = 0; b < WB; ++b) acc[i][b] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  struct Tile {
    float4 a[4][RB], w[4][WB], g[NORM ? 4 : 1];
  };
  // the four 16-k steps of 64-k tile t; A past K is zero (W is padded)
  auto load = [&](int t, Tile& x) __attribute__((always_inline)) {
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      const int k = t * kWTile + 16 * s;
#pragma unroll
      for (int b = 0; b < WB; ++b) x.w[s][b] = *(const float4*)(wp[b] + (long)t * kWTileElts + 16 * s);
      if constexpr (NORM) x.g[s] = k + 4 * h < K ? *(const float4*)(gain + k + 4 * h) : make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
      for (int i = 0; i < RB; ++i) {
        const int ke = k + 4 * h;
        if constexpr (VEC) {
          x.a[s][i] = ke < K ? *(const float4*)(ap[i] + k) : make_float4(0.f, 0.f, 0.f, 0.f);
        } else {
          x.a[s][i] = make_float4(ke < K ? ap[i][k] : 0.f, ke + 1 < K ? ap[i][k + 1] : 0.f,
                                  ke + 2 < K ? ap[i][k + 2] : 0.f, ke + 3 < K ? ap[i][k + 3] : 0.f);
        }
      }
    }
  };
  float ss[RB];  // NORM: this lane's share of its rows' sums of squares
#pragma unroll
  for (int i = 0; i < RB; ++i) ss[i] = 0.f;
  auto mul = [&](Tile& x) __attribute__((always_inline)) {
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      if constexpr (NORM) {
#pragma unroll
        for (int i = 0; i < RB; ++i) {
          float4& v = x.a[s][i];
          ss[i] = fmaf(v.x, v.x, fmaf(v.y, v.y, fmaf(v.z, v.z, fmaf(v.w, v.w, ss[i]))));
          v = make_float4(v.x * x.g[s].x, v.y * x.g[s].y, v.z * x.g[s].z, v.w * x.g[s].w);
        }
      }
      auto step = [&](auto pick) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < RB; ++i)
#pragma unroll
          for (int b = 0; b < WB; ++b)
            acc[i][b] = __builtin_amdgcn_mfma_f32_16x16x4f32(pick(x.a[s][i]), pick(x.w[s][b]), acc[i][b], 0, 0, 0);
      };
      step([](const float4& v) { return v.x; });
      step([](const float4& v) { return v.y; });
      step([](const float4& v) { return v.z; });
      step([](const float4& v) { return v.w; });
    }
  };
  Tile x0, x1;
  int t = t0;
  if (t < t1) load(t, x0);
  for (; t + 1 < t1; t += 2) {
    load(t + 1, x1);
    mul(x0);
    if (t + 2 < t1) load(t + 2, x0);
    mul(x1);
  }
  if (t < t1) mul(x0);

  // acc[i][b][e] is row m0 + 16 i + 4 h + e, column r16 of block b
  auto store = [&](int i, int cb, int e, float g, float u) __attribute__((always_inline)) {
    const int row = m0 + 16 * i + 4 * h + e, col = c0 + 16 * cb + r16;
    const int ldc = EPI == 2 ? N / 2 : N;
    if (row >= M || col >= ldc) return;
    const long idx = (long)row * ldc + col;
    float v = g;
    if constexpr (EPI == 1) v += ld_elt<TR>(R, idx);
    if constexpr (EPI == 2) v = silu_f(g) * u;
    st_elt<TC>(C, idx, v);
  };
  if constexpr (KSPLIT) {
    __shared__ f32x4_t part[4][RB * WB][64];
#pragma unroll
    for (int i = 0; i < RB; ++i)
#pragma unroll
      for (int b = 0; b < WB; ++b) part[wave][i * WB + b][lane] = acc[i][b];
    __shared__ float s_ss[4][NORM ? 16 * RB : 1];
    if constexpr (NORM) {
#pragma unroll
      for (int i = 0; i < RB; ++i) {
        ss[i] += __shfl_xor(ss[i], 16);
        ss[i] += __shfl_xor(ss[i], 32);
        if (h == 0) s_ss[wave][16 * i + r16] = ss[i];
      }
    }
    __syncthreads();
    // wave w finishes output block w, w + 4, ...
    constexpr int PB = EPI == 2 ? 2 : 1;
    for (int o = wave; o < RB * CB; o += 4) {
      f32x4_t sum[PB];
#pragma unroll
      for (int p = 0; p < PB; ++p) {
        sum[p] = part[0][o * PB + p][lane];
        for (int w = 1; w < 4; ++w) sum[p] += part[w][o * PB + p][lane];
      }
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        float inv = 1.f;
        if constexpr (NORM) {
          const int r = 16 * (o / CB) + 4 * h + e;
          inv = 1.0f / sqrtf(((s_ss[0][r] + s_ss[1][r]) + (s_ss[2][r] + s_ss[3][r])) / (float)K + eps);
        }
        store(o / CB, o % CB, e, sum[0][e] * inv, sum[PB - 1][e] * inv);
      }
    }
  } else {
#pragma unroll
    for (int i = 0; i < RB; ++i)
#pragma unroll
      for (int cb = 0; cb < CB; ++cb)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          if constexpr (EPI == 2) store(i, cb, e, acc[i][2 * cb][e], acc[i][2 * cb + 1][e]);
          else store(i, cb, e, acc[i][cb][e], 0.f);
        }
  }
}

// ==================================================================== launch
int compute_units() {
  static const int n = [] {
    int dev = 0, v = 0;
    if (hipGetDevice(&dev) != hipSuccess || hipDeviceGetAttribute(&v, hipDeviceAttributeMultiprocessorCount, dev) !=
                                                 hipSuccess || v <= 0)
      return 256;
    return v;
  }();
  return n;
}

// The tile kernel's shapes. `start` and `stage` are microseconds of one
// workgroup alone on its compute unit: prologue + epilogue, and one 64-k
// stage. Least-squares fits over the 8B and 70B layers' GEMMs at 80 to 4096
// rows and 1 to 4 K splits, weights cold in every cache (rms error 7-16%; the
// shape and splits chosen are within 1% of the best measured on average, 14%
// at worst). Per output element a larger tile is cheaper (256x256: 1.26 us per
// stage for four 128x128 tiles' work at 0.47 each) but fills fewer compute units.
struct TileCfg {
  int qm, qn;  // 64 qm x 64 qn outputs per workgroup
  float start, stage;
};
constexpr TileCfg kTileCfgs[] = {
    {4, 4, 13.7f, 1.260f}, {3, 4, 10.7f, 1.127f}, {2, 4, 10.3f, 0.735f}, {4, 2, 10.6f, 0.715f},
    {3, 2, 7.6f, 0.571f},  {2, 2, 7.4f, 0.466f},  {2, 1, 6.0f, 0.326f},  {1, 1, 4.0f, 0.250f},
};
constexpr int kTileCfgCount = sizeof(kTileCfgs) / sizeof(kTileCfgs[0]);

// Cost in microseconds of a tile-kernel launch: rounds of workgroups over the
// compute units (one resident per unit), the weight stream (5 TB/s) that the
// rounds cannot beat and only partly hide, and the split partials (fp32,
// written, then read by the consumer, ~6 TB/s). M counts in whole 64-row
// blocks, so that the choice is constant between multiples of 64.
static double tile_cost(const TileCfg& t, int M, int N, int K, int S) {
  const long cu = compute_units(), rows = (M + 63) / 64 * 64;
  const long wgs = (long)((M + 64 * t.qm - 1) / (64 * t.qm)) * (N / (64 * t.qn)) * S;
  const int T = K / tile::BK;
  const double work = (double)((wgs + cu - 1) / cu) * (t.start + t.stage * ((T + S - 1) / S));
  const double stream = (double)N * K * 2.0 / 5.0e6;
  return std::max(work, stream) + 0.3 * std::min(work, stream) + (S > 1 ? (double)S * rows * N * 8.0 / 6.0e6 : 0.0);
}

// The most K splits a tile launch may take: 4, of at least 16 stages each, and no
// more of them than fill one round of 256x256 tiles (two above 2048 rows, where an
// unsplit launch ends in a nearly empty round: down at 2257 rows 295 us unsplit,
// 287 with its reduce in two splits); that bounds the partials at 256 KiB per tile
// and split.
static int tile_most_splits(int M, int N, int K) {
  const long tiles256 = (long)((M + 255) / 256) * (N / 256), fit = (M > 2048 ? 2 : 1) * compute_units();
  int S = 1;
  while (S < 4 && K / tile::BK / (S + 1) >= 16 && tiles256 * (S + 1) <= fit) ++S;
  return S;
}

// The cheapest tile shape and, up to max_splits, K splits. SwiGLU pairs a
// gate and an up block within a wave, so its tiles are at least 128 wide. The
// outputs of an unsplit launch do not depend on the tile shape: each is one
// chain of the same MFMAs over K.
TilePlan gemm_tile_plan(int M, int N, int K, int max_splits, bool swiglu, double* cost) {
  TilePlan best{0, 1};
  if (cost) *cost = 0;
  if (M <= skinny::MAXM || N % 256 || K % tile::BK) return best;
  double best_cost = 0;
  for (int S = 1, most = std::min(max_splits, tile_most_splits(M, N, K)); S <= most; ++S) {
    for (int i = 0; i < kTileCfgCount; ++i) {
      if (swiglu && kTileCfgs[i].qn % 2) continue;
      const double c = tile_cost(kTileCfgs[i], M, N, K, S);
      if ((S == 1 && i == 0) || c < best_cost) best = TilePlan{i, S}, best_cost = c;
    }
  }
  if (cost) *cost = best_cost;
  return best;
}

// A launch of several rounds whose last is nearly empty costs less in two
// parts: as many columns as whole rounds of a large tile take, then the rest in
// the shape that is cheapest for them. Returns the first part's columns (0: one
// launch) with both shapes. Taken where the cost model promises 6%, another
// launch's 4 us included (us, one launch -> two): N 28672, K 4096 at 700 rows 169
// -> 151, at 1800 378 -> 356, at 3000 555 -> 535; N 57344, K 8192 at 1000 747 ->
// 702; N 10240, K 8192 at 2048 296 -> 268; N 6144, K 4096 at 3500 144 -> 139.
// Where it promised 4 to 5% it gave 1 or 2, once -2. Beside another stream's
// attention it loses (mixed step of 4 x 512 + 32 rows 1074 -> 1081).
static int tile_columns(int M, int N, int K, bool swiglu, const TilePlan& whole, TilePlan* first, TilePlan* rest) {
  const long cu = compute_units();
  auto wgs = [&](const TileCfg& t, int n) { return (long)((M + 64 * t.qm - 1) / (64 * t.qm)) * (n / (64 * t.qn)); };
  if (whole.s != 1 || wgs(kTileCfgs[whole.cfg], N) <= cu) return 0;
  double best = tile_cost(kTileCfgs[whole.cfg], M, N, K, 1) / 1.06;
  int cols = 0;
  for (int i = 0; i < 4; ++i) {
    const TileCfg& t = kTileCfgs[i];
    const long tiles_m = (M + 64 * t.qm - 1) / (64 * t.qm);
    const int n = (int)(wgs(t, N) / cu * cu / tiles_m * (64 * t.qn) / 256 * 256);
    if (n <= 0 || n >= N) continue;
    double c;
    const TilePlan r = gemm_tile_plan(M, N - n, K, 1, swiglu, &c);
    c += tile_cost(t, M, n, K, 1) + 4.0;
    if (c < best) best = c, cols = n, *first = TilePlan{i, 1}, *rest = r;
  }
  return cols;
}

int gemm_tile_splits(int M, int N, int K) { return gemm_tile_plan(M, N, K, 4, false).s; }

TilePartials::TilePartials(int N, int K, int max_rows) : n_(N), k_(K) {
  if (N <= 0 || N % 256 || K % tile::BK) return;
  // past as many rows nothing is split: two splits would take more than two rounds
  const long last = std::min<long>(max_rows, 256L * (compute_units() / (N / 256)));
  rows_.assign(2, 0);  // up to 64 rows: the skinny path
  for (int m = 128; m <= last; m += 64) {
    const int S = gemm_tile_splits(m, N, K);
    rows_.push_back(std::max(rows_.back(), S > 1 ? S * m : 0));
  }
}

size_t TilePartials::bytes(int max_rows) const {
  if (rows_.empty() || max_rows <= skinny::MAXM) return 0;
  int rows = rows_[std::min<size_t>(max_rows / 64, rows_.size() - 1)];
  if (max_rows % 64)
    if (const int S = gemm_tile_splits(max_rows, n_, k_); S > 1) rows = std::max(rows, S * max_rows);
  return (size_t)rows * n_ * sizeof(float);
}

// Tile rows walked per group (see the kernel). Few rows (up to ~2300): groups
// of equal size of at most ~1280 rows, so that the workgroups sharing a
// weight column run together and no short group trails; more rows: 8 tile
// rows of 256 on wide outputs (more W reuse per XCD), 4 on narrow ones.
static int tile_group(int M, int N, int qm) {
  const int tiles_m = (M + 64 * qm - 1) / (64 * qm);
  if (M <= 2304) {
    const int groups = (tiles_m * 64 * qm + 1279) / 1280;
    return (tiles_m + groups - 1) / groups;
  }
  return std::max(1, (N / 256 >= 64 ? 2048 : 1024) / (64 * qm));
}

// The layer's launches take any shape; the remaining type combinations
// (single-op calls) run 256x256 tiles only.
template <int EPI, typename TR, typename TC>
constexpr bool kTileAllShapes = (EPI == 0 && std::is_same<TR, float>::value) ||
                                (EPI == 1 && !std::is_same<TR, TC>::value) ||
                                (EPI == 2 && std::is_same<TC, bf16_t>::value);

#define PS_TILE_EXTERN(QM, QN, NS, NT, EPI, TR, TC)                                                                     \
  extern template int launch_tile_g<QM, QN, NS, NT, EPI, TR, TC>(int, int, int, int, const void*, const void*,         \
                                                                 const void*, void*, hipStream_t, int, int);
PS_TILE_INSTANCES(PS_TILE_EXTERN)
#undef PS_TILE_EXTERN

template <int EPI, typename TR, typename TC>
static int launch_tile_cols(int M, int N, int cols, int K, TilePlan pl, const void* A, const void* W, const void* R,
                            void* C, hipStream_t st) {
  const int group = tile_group(M, cols, kTileCfgs[pl.cfg].qm);
  // One tile row: weight loads with the non-temporal hint (see the kernel).
  // Two rows of 192x256 or 256x256 tiles gain too (us, N 57344, K 8192: 300
  // rows 358 -> 348, 512 rows 418 -> 401; N 28672, K 4096 at 389 102 -> 99).
  // Otherwise workgroups that share weights drift apart where the last tile row
  // is short, and the hint costs up to 20% (N 4096, K 14336 at 300 rows: 70, with
  // it 88), and from four rows on it gives nothing or loses 1 to 7%.
  const TileCfg& tc = kTileCfgs[pl.cfg];
  const bool nt = M <= 64 * tc.qm * (tc.qm >= 3 && tc.qn == 4 ? 2 : 1);
#define PS_TILE_GO(QM, QN, NS, NT) launch_tile_g<QM, QN, NS, NT, EPI, TR, TC>(M, N, cols, K, A, W, R, C, st, pl.s, group)
#define PS_TILE_GO_NT(QM, QN, NS) (nt ? PS_TILE_GO(QM, QN, NS, true) : PS_TILE_GO(QM, QN, NS, false))
  if constexpr (kTileAllShapes<EPI, TR, TC>) {
    switch (pl.cfg) {
      case 0: return PS_TILE_GO_NT(4, 4, 2);
      case 1: return PS_TILE_GO_NT(3, 4, 2);
      case 2: return PS_TILE_GO_NT(2, 4, 3);
      case 3: return PS_TILE_GO_NT(4, 2, 3);
      case 4: return PS_TILE_GO_NT(3, 2, 3);
      case 5: return PS_TILE_GO_NT(2, 2, 4);
      default: break;
    }
    if constexpr (EPI != 2) {
      if (pl.cfg == 6) return PS_TILE_GO_NT(2, 1, 6);
      if (pl.cfg == 7) return PS_TILE_GO(1, 1, 5, false);  // M > 64: two tile rows at least
    }
    return -1;
  } else {
    return PS_TILE_GO(4, 4, 2, false);
  }
#undef PS_TILE_GO_NT
#undef PS_TILE_GO
}

template <int EPI, typename TR, typename TC>
static int launch_tile(int M, int N, int K, TilePlan pl, const void* A, const void* W, const void* R, void* C,
                       hipStream_t st, bool beside = false) {
  if constexpr (!kTileAllShapes<EPI, TR, TC>) {
    return launch_tile_cols<EPI, TR, TC>(M, N, N, K, TilePlan{0, pl.s}, A, W, R, C, st);
  } else {
    TilePlan a, b;
    const int n = beside ? 0 : tile_columns(M, N, K, EPI == 2, pl, &a, &b);
    if (n == 0) return launch_tile_cols<EPI, TR, TC>(M, N, N, K, pl, A, W, R, C, st);
    if (launch_tile_cols<EPI, TR, TC>(M, N, n, K, a, A, W, R, C, st)) return -1;
    const bf16_t* w = (const bf16_t*)W + (long)(n / 64) * (K / 64) * kWTileElts;
    const void* r = R ? (const TR*)R + n : nullptr;
    return launch_tile_cols<EPI, TR, TC>(M, N, N - n, K, b, A, w, r, (TC*)C + (EPI == 2 ? n / 2 : n), st);
  }
}

int launch_gemm_tile_split(int M, int N, int K, int S, const void* A, const void* W, float* part, hipStream_t st) {
  if (M <= 0 || S < 1 || N % 256 || K % tile::BK || K / tile::BK < S) return -1;
  TilePlan pl = gemm_tile_plan(M, N, K, 4, false);
  if (pl.s != S) return -1;
  return launch_tile<0, float, float>(M, N, K, pl, A, W, nullptr, part, st);
}

template <int EPI, typename TR, typename TC>
static int launch_reduce(int M, int N, int S, const float* part, const void* R, void* C, hipStream_t st);

int launch_split_residual(int r_dt, int c_dt, int M, int N, int S, const float* part, const void* R, void* C,
                          hipStream_t st) {
  if (M == 0) return 0;
  if (r_dt == 0 && c_dt == 1) return launch_reduce<1, float, bf16_t>(M, N, S, part, R, C, st);
  if (r_dt == 1 && c_dt == 1) return launch_reduce<1, bf16_t, bf16_t>(M, N, S, part, R, C, st);
  if (r_dt == 1 && c_dt == 0) return launch_reduce<1, bf16_t, float>(M, N, S, part, R, C, st);
  if (r_dt == 0 && c_dt == 0) return launch_reduce<1, float, float>(M, N, S, part, R, C, st);
  return -1;
}

template <typename TR, typename TC>
__global__ __launch_bounds__(256) void gemm_reduce_residual4_kernel(const float* __restrict__ part,
                                                                    const TR* __restrict__ R, TC* __restrict__ C,
                                                                    long n4, long mn, int S) {
  for (long e = (long)blockIdx.x * 256 + threadIdx.x; e < n4; e += (long)gridDim.x * 256) {
    float4 v = ((const float4*)part)[e];
    for (int s = 1; s < S; ++s) {
      const float4 p = ((const float4*)(part + s * mn))[e];
      v.x += p.x, v.y += p.y, v.z += p.z, v.w += p.w;
    }
    if constexpr (std::is_same<TR, float>::value) {
      const float4 r = ((const float4*)R)[e];
      v.x += r.x, v.y += r.y, v.z += r.z, v.w += r.w;
    } else {
      const uint2 r = ((const uint2*)R)[e];
      v.x += __uint_as_float(r.x << 16), v.y += __uint_as_float(r.x & 0xffff0000u);
      v.z += __uint_as_float(r.y << 16), v.w += __uint_as_float(r.y & 0xffff0000u);
    }
    if constexpr (std::is_same<TC, float>::value)
      ((float4*)C)[e] = v;
    else
      ((uint2*)C)[e] = uint2{pack_bf2(v.x, v.y), pack_bf2(v.z, v.w)};
  }
}

template <int EPI, typename TR, typename TC>
static int launch_reduce(int M, int N, int S, const float* part, const void* R, void* C, hipStream_t st) {
  const long total = (EPI == 2) ? (long)M * (N / 2) : (long)M * N;
  if constexpr (EPI == 1) {
    auto al = [](const void* p, uintptr_t a) { return ((uintptr_t)p & (a - 1)) == 0; };
    if (N % 4 == 0 && al(part, 16) && al(R, 4 * sizeof(TR)) && al(C, 4 * sizeof(TC))) {
      const long n4 = total / 4;
      const int blocks = (int)std::min<long>((n4 + 255) / 256, 8192);
      hipLaunchKernelGGL((gemm_reduce_residual4_kernel<TR, TC>), dim3(blocks), dim3(256), 0, st, part, (const TR*)R,
                         (TC*)C, n4, total, S);
      return 0;
    }
  }
  int blocks = (int)std::min<long>((total + 255) / 256, 4096);
  hipLaunchKernelGGL((gemm_reduce_kernel<EPI, TR, TC>), dim3(blocks), dim3(256), 0, st, part, (const TR*)R, (TC*)C,
                     M, N, S);
  return 0;
}

// Skinny launch plan: WN 64-row blocks per workgroup and S K-splits. Two
// blocks per workgroup halve the activation traffic per weight byte and win
// whenever the grid still reaches ~160 workgroups; otherwise one block. The
// split count is the largest that keeps the grid within one round of 256
// workgroups, at most 8, while each split keeps at least 16 stages (shorter
// splits lose more to ring fill and drain than they gain in parallelism, and
// add partial-sum traffic); splits are near-equal stage ranges, so any count
// works. Chosen from a sweep of both widths and 1..8 splits over the 8B and
// 70B decode shapes at M = 32 and 64, reduction included.
static int skinny_splits_for(int tiles, int K, int target) {
  using namespace skinny;
  const int stages = K / KS;
  int S = std::max(1, std::min(8, target / tiles));
  while (S > 1 && stages / S < 16) --S;
  return S;
}

//
// Four blocks per workgroup (S 1) where two would take more than one round of
// the compute units: at least 160 workgroups that fit seven eighths of them (us,
// two -> four blocks: N 57344, K 8192 at 1 row 134.7 -> 130.9, at 64 147 -> 133;
// N 40960, K 8192 at 8 rows 116 -> 99; N 49152, K 4096 at 64 72 -> 62), and above
// that from 33 rows on, where halving the activation reads pays (N 128256, K
// 4096 at 64 rows 196 -> 176; but at 8 rows 157 -> 163, N 65536, K 8192 155 -> 158).
SkinnyPlan gemm_skinny_plan(int M, int N, int K) {
  if (N % 256 == 0 && N / 128 > 256 && N / 256 >= 160 && (N / 256 <= 224 || M > 32)) return {4, 1};
  if (N % 128 == 0) {
    const int S = skinny_splits_for(N / 128, K, 256);
    if ((N / 128) * S >= 160) return {2, S};
  }
  return {1, skinny_splits_for(N / 64, K, 256)};
}

template <int MB, int WN, int EPI, typename TR, typename TC, bool DIRECT>
static int launch_skinny_k(int M, int N, int K, int S, const void* A, const void* W, float* part, const void* R,
                           void* C, hipStream_t st) {
  constexpr size_t lds = skinny::lds_bytes<MB, WN>();
  static const hipError_t attr = hipFuncSetAttribute(
      (const void*)gemm_skinny_kernel<MB, WN, EPI, TR, TC, DIRECT>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  if (attr != hipSuccess) return -1;
  hipLaunchKernelGGL((gemm_skinny_kernel<MB, WN, EPI, TR, TC, DIRECT>), dim3(N / (64 * WN), S), dim3(skinny::NT), lds,
                     st, (const bf16_t*)A, (const bf16_t*)W, part, (const TR*)R, (TC*)C, M, N, K, S);
  return 0;
}

template <int MB, int WN, int EPI, typename TR, typename TC>
static int launch_skinny_wn(int M, int N, int K, int S, const void* A, const void* W, float* part, const void* R,
                            void* C, hipStream_t st) {
  if constexpr (EPI != 2 || WN == 2) {
    if (S == 1) return launch_skinny_k<MB, WN, EPI, TR, TC, true>(M, N, K, 1, A, W, part, R, C, st);
  }
  if (launch_skinny_k<MB, WN, EPI, TR, TC, false>(M, N, K, S, A, W, part, R, C, st)) return -1;
  return launch_reduce<EPI, TR, TC>(M, N, S, part, R, C, st);
}

template <int MB, int EPI, typename TR, typename TC>
static int launch_skinny_mb(int M, int N, int K, SkinnyPlan pl, const void* A, const void* W, float* part,
                            const void* R, void* C, hipStream_t st) {
  if (pl.wn == 4) return launch_skinny_k<MB, 4, EPI, TR, TC, true>(M, N, K, 1, A, W, part, R, C, st);
  if (pl.wn == 2) return launch_skinny_wn<MB, 2, EPI, TR, TC>(M, N, K, pl.s, A, W, part, R, C, st);
  return launch_skinny_wn<MB, 1, EPI, TR, TC>(M, N, K, pl.s, A, W, part, R, C, st);
}

template <int EPI, typename TR, typename TC>
static int launch_skinny_plan(int M, int N, int K, SkinnyPlan pl, const void* A, const void* W, float* part,
                              const void* R, void* C, hipStream_t st) {
  if ((pl.wn != 1 && pl.wn != 2 && (pl.wn != 4 || pl.s != 1)) || N % (64 * pl.wn) != 0 || pl.s < 1 || K / skinny::KS < pl.s) return -1;
  switch ((M + 15) / 16) {
    case 1: return launch_skinny_mb<1, EPI, TR, TC>(M, N, K, pl, A, W, part, R, C, st);
    case 2: return launch_skinny_mb<2, EPI, TR, TC>(M, N, K, pl, A, W, part, R, C, st);
    case 3: return launch_skinny_mb<3, EPI, TR, TC>(M, N, K, pl, A, W, part, R, C, st);
    case 4: return launch_skinny_mb<4, EPI, TR, TC>(M, N, K, pl, A, W, part, R, C, st);
    default: return -1;
  }
}

template <int EPI, typename TR, typename TC>
static int launch_skinny(int M, int N, int K, const void* A, const void* W, float* part, const void* R, void* C,
                         hipStream_t st) {
  return launch_skinny_plan<EPI, TR, TC>(M, N, K, gemm_skinny_plan(M, N, K), A, W, part, R, C, st);
}

// `norm`: the input rows are normalised in the kernel (gemm_f32_norm_ok)
struct F32Norm {
  const float* gain;
  float eps;
  UploadJob up;
};
template <int RB, int CB, bool KSPLIT, int EPI, typename TR, typename TC>
static int launch_f32_shape(int M, int N, int K, const void* A, const void* W, const void* R, void* C, hipStream_t st,
                            const F32Norm* norm = nullptr) {
  constexpr int MW = KSPLIT ? 1 : 2;
  const int cols = EPI == 2 ? N / 2 : N;
  dim3 grid((cols + 16 * CB * MW - 1) / (16 * CB * MW), (M + 16 * RB * MW - 1) / (16 * RB * MW));
  auto go = [&](auto vec, auto nc) {
    const F32Norm n = norm ? *norm : F32Norm{nullptr, 0.f, UploadJob{}};
    grid.x += n.up.blocks;
    hipLaunchKernelGGL((gemm_f32_kernel<RB, CB, KSPLIT, decltype(vec)::value, decltype(nc)::value, EPI, TR, TC>), grid,
                       dim3(f32g::NT), 0, st, (const float*)A, (const float*)W, (const TR*)R, (TC*)C, M, N, K, n.gain,
                       n.eps, n.up);
  };
  if constexpr (KSPLIT && EPI != 1) {
    if (norm) {
      go(std::true_type{}, std::true_type{});
      return 0;
    }
  }
  if (norm) return -1;
  if (K % 4 == 0) go(std::true_type{}, std::false_type{});
  else go(std::false_type{}, std::false_type{});
  return 0;
}

// 128 x 128 tiles (64 x 64 per wave) where they reach half the compute units
// (1024 x 1024 x 1024 in 32 x 32 tiles: 40 us against 64 tiles of 128 x 128 that
// leave three quarters idle); else K split over the waves.
static bool f32_large(int epi, int M, int N) {
  const int cols = epi == 2 ? N / 2 : N;
  const long tiles = (long)((M + 127) / 128) * ((cols + (epi == 2 ? 63 : 127)) / (epi == 2 ? 64 : 128));
  return tiles >= compute_units() / 2;
}

template <int EPI, typename TR, typename TC>
static int launch_f32(int M, int N, int K, const void* A, const void* W, const void* R, void* C, hipStream_t st,
                      const F32Norm* norm = nullptr) {
  if (f32_large(EPI, M, N)) return launch_f32_shape<4, EPI == 2 ? 2 : 4, false, EPI, TR, TC>(M, N, K, A, W, R, C, st, norm);
  // 16 rows at a time for decode-sized M
  if (M <= 16) return launch_f32_shape<1, 1, true, EPI, TR, TC>(M, N, K, A, W, R, C, st, norm);
  return launch_f32_shape<2, EPI == 2 ? 1 : 2, true, EPI, TR, TC>(M, N, K, A, W, R, C, st, norm);
}

bool gemm_f32_norm_ok(int epi, int M, int N, int K) {
  return epi != 1 && M > 0 && K % 4 == 0 && (epi != 2 || N % 64 == 0) && !f32_large(epi, M, N);
}

int launch_gemm_f32_norm(int epi, int M, int N, int K, const float* x, const float* gain, float eps, const float* W,
                         float* C, hipStream_t st, const UploadJob* up) {
  if (!gemm_f32_norm_ok(epi, M, N, K)) return -1;
  const F32Norm n{gain, eps, up ? *up : UploadJob{}};
  if (epi == 0) return launch_f32<0, float, float>(M, N, K, x, W, nullptr, C, st, &n);
  return launch_f32<2, float, float>(M, N, K, x, W, nullptr, C, st, &n);
}

size_t gemm_workspace_bytes(int dtype, int M, int N, int K) {
  if (dtype != 1 || M > skinny::MAXM) return 0;
  return (size_t)gemm_skinny_plan(M, N, K).s * M * N * sizeof(float);
}

// Dispatch on (dtype, r_dtype, c_dtype, epilogue) and on M.
int launch_gemm(int dtype, int r_dt, int c_dt, int epi, int M, int N, int K, const void* A, const void* W,
                const void* R, void* C, void* ws, size_t ws_bytes, hipStream_t st, bool beside) {
  if (M == 0) return 0;
  if (dtype == 0) {
    if (N % 64 != 0 && epi == 2) return -1;
#define F32_CASE(E, TR_, TC_, rd, cd) \
  if (epi == E && r_dt == rd && c_dt == cd) return launch_f32<E, TR_, TC_>(M, N, K, A, W, R, C, st);
    F32_CASE(0, float, float, 0, 0)
    F32_CASE(0, float, float, 1, 0)
    F32_CASE(1, float, float, 0, 0)
    F32_CASE(2, float, float, 0, 0)
    F32_CASE(2, float, float, 1, 0)
#undef F32_CASE
    return -1;
  }
  if (K % 64 != 0) return -1;
  if (M <= skinny::MAXM && N % 64 == 0) {
    if (ws_bytes < gemm_partials_bytes(dtype, epi, M, N, K)) return -2;
    float* part = (float*)ws;
#define SK_CASE(E, TR_, TC_, rd, cd) \
  if (epi == E && r_dt == rd && c_dt == cd) return launch_skinny<E, TR_, TC_>(M, N, K, A, W, part, R, C, st);
    SK_CASE(0, float, bf16_t, 0, 1)
    SK_CASE(0, float, bf16_t, 1, 1)
    SK_CASE(0, float, float, 0, 0)
    SK_CASE(0, float, float, 1, 0)
    SK_CASE(1, bf16_t, float, 1, 0)
    SK_CASE(1, float, bf16_t, 0, 1)
    SK_CASE(1, bf16_t, bf16_t, 1, 1)
    SK_CASE(1, float, float, 0, 0)
    SK_CASE(2, float, bf16_t, 0, 1)
    SK_CASE(2, float, bf16_t, 1, 1)
    SK_CASE(2, float, float, 0, 0)
#undef SK_CASE
    return -1;
  }
  if (N % 256 != 0) return -1;
#define TILE_CASE(E, TR_, TC_, rd, cd) \
  if (epi == E && r_dt == rd && c_dt == cd)  \
    return launch_tile<E, TR_, TC_>(M, N, K, gemm_tile_plan(M, N, K, 1, E == 2), A, W, R, C, st, beside);
  TILE_CASE(0, float, bf16_t, 0, 1)
  TILE_CASE(0, float, bf16_t, 1, 1)
  TILE_CASE(0, float, float, 0, 0)
  TILE_CASE(0, float, float, 1, 0)
  TILE_CASE(1, bf16_t, float, 1, 0)
  TILE_CASE(1, float, bf16_t, 0, 1)
  TILE_CASE(1, bf16_t, bf16_t, 1, 1)
  TILE_CASE(1, float, float, 0, 0)
  TILE_CASE(2, float, bf16_t, 0, 1)
  TILE_CASE(2, float, bf16_t, 1, 1)
  TILE_CASE(2, float, float, 0, 0)
#undef TILE_CASE
  return -1;
}

// launch_gemm, except that a decode-sized bf16 GEMM whose plan splits K in
// 2, 3, 4 or 8 stops at the split partials (fp32 [S][M][N] at the head of ws,
// summed in split order by the consumer, which fuses the reduction with its
// own work); *splits = S then, else 1 and C holds the result.
int launch_gemm_split(int dtype, int r_dt, int c_dt, int epi, int M, int N, int K, const void* A, const void* W,
                      const void* R, void* C, void* ws, size_t ws_bytes, hipStream_t st, int* splits, bool beside) {
  *splits = 1;
  if (dtype == 1 && M > 0 && M <= skinny::MAXM && N % 64 == 0 && K % 64 == 0 && epi != 2) {
    const SkinnyPlan pl = gemm_skinny_plan(M, N, K);
    if (pl.s == 2 || pl.s == 3 || pl.s == 4 || pl.s == 8) {  // the split counts the fused consumers take
      if (ws_bytes < gemm_workspace_bytes(dtype, M, N, K)) return -2;
      *splits = pl.s;
      float* part = (float*)ws;
      // the partial kernel's output does not depend on the epilogue or the
      // output types (only its weight-row mapping does, for SwiGLU)
      auto go = [&](auto mbc) {
        constexpr int MB = decltype(mbc)::value;
        if (pl.wn == 2) return launch_skinny_k<MB, 2, 0, float, float, false>(M, N, K, pl.s, A, W, part, R, C, st);
        return launch_skinny_k<MB, 1, 0, float, float, false>(M, N, K, pl.s, A, W, part, R, C, st);
      };
      switch ((M + 15) / 16) {
        case 1: return go(std::integral_constant<int, 1>{});
        case 2: return go(std::integral_constant<int, 2>{});
        case 3: return go(std::integral_constant<int, 3>{});
        default: return go(std::integral_constant<int, 4>{});
      }
    }
  }
  return launch_gemm(dtype, r_dt, c_dt, epi, M, N, K, A, W, R, C, ws, ws_bytes, st, beside);
}

// Bytes of split-K partials a bf16 launch actually writes: 0 for the tile
// path and for skinny launches that apply their epilogue in the kernel.
size_t gemm_partials_bytes(int dtype, int epi, int M, int N, int K) {
  if (dtype != 1 || M <= 0 || M > skinny::MAXM || N % 64 != 0 || K % 64 != 0) return 0;
  const SkinnyPlan pl = gemm_skinny_plan(M, N, K);
  if (pl.s == 1 && (epi != 2 || pl.wn >= 2)) return 0;
  return (size_t)pl.s * M * N * sizeof(float);
}

// ------------------------------------------------------------ static scratch
// Split-K partials for callers that cannot allocate device memory: a
// file-scope device array, one copy on every GPU the library runs on, kept
// until the process ends. In host code `scratch` names a host-side stand-in,
// not a device address, so host code never passes it to a kernel or a copy:
// gemm_static_scratch() returns the device address of the current GPU's
// copy, looked up once per device with hipGetSymbolAddress.
static __device__ __align__(256) uint8_t scratch[kGemmStaticScratchBytes];

namespace {
constexpr int kMaxScratchDevices = 64;
std::mutex g_scratch_mu;
void* g_scratch_ptr[kMaxScratchDevices] = {};
}  // namespace

hipError_t gemm_static_scratch(void** out) {
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= kMaxScratchDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (!g_scratch_ptr[dev]) {
    void* p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    g_scratch_ptr[dev] = p;
  }
  *out = g_scratch_ptr[dev];
  return hipSuccess;
}

}  // namespace ps

namespace ps {
// Host-side mirror of launch_gemm's dispatch conditions: 0 if supported.
int gemm_check(int dtype, int epi, int M, int N, int K) {
  if (M < 0 || N <= 0 || K <= 0) return -1;
  if (epi == 2 && N % (2 * kGateUpBlock) != 0) return -1;
  if (dtype == 0) return 0;
  if (dtype != 1 || K % 64 != 0 || K >= (1 << 21)) return -1;  // 32-bit byte offsets per 256-row tile
  if (M <= skinny::MAXM && N % 64 == 0) return 0;
  return (N % 256 == 0) ? 0 : -1;
}
}  // namespace ps
