// Device helpers shared by the GEMM kernels, and the tile GEMM (M > 64): a
// template over its workgroup tile and LDS ring, instantiated in
// k_gemm_tile_*.hip and chosen per launch by gemm_tile_plan (k_gemm.hip).
#pragma once
#include "common.h"
#include "launch.h"

#include <type_traits>

namespace ps {

__device__ __forceinline__ float silu_f(float x) { return x / (1.f + expf(-x)); }
// silu on the hardware exp2 and reciprocal (v_exp_f32, v_rcp_f32): a few
// fp32 ulp, far below the bf16 rounding of the GEMM operands; four vector
// instructions instead of the ~30 of expf and an IEEE divide, which matter
// in an epilogue that no matrix work overlaps. x -> -inf gives -0, x -> inf
// gives x.
__device__ __forceinline__ float silu_fast(float x) {
  return x * __builtin_amdgcn_rcpf(1.f + __builtin_amdgcn_exp2f(x * -1.4426950408889634f));
}

template <typename T> __device__ __forceinline__ float ld_elt(const T* p, long i);
template <> __device__ __forceinline__ float ld_elt<float>(const float* p, long i) { return p[i]; }
template <> __device__ __forceinline__ float ld_elt<bf16_t>(const bf16_t* p, long i) { return bf2f(p[i]); }
template <typename T> __device__ __forceinline__ void st_elt(T* p, long i, float v);
template <> __device__ __forceinline__ void st_elt<float>(float* p, long i, float v) { p[i] = v; }
template <> __device__ __forceinline__ void st_elt<bf16_t>(bf16_t* p, long i, float v) { p[i] = f2bf(v); }

// ================================================================== helpers
// One 16-byte global->LDS fill per lane through a buffer resource
// (buffer_load_dwordx4 ... lds): a wave instruction fills 1 KiB of LDS, lane
// l landing at +16 l; `voffset` is the lane's byte offset from the resource
// base. The compiler counts this form on vmcnt alone, so LDS reads issued
// around it keep exact lgkmcnt waits (around the FLAT global_load_lds form
// it waits for every outstanding LDS read before each use of a fragment).
__device__ __forceinline__ void load_lds16_buf(__amdgpu_buffer_rsrc_t r, uint32_t voffset, bf16_t* lds) {
  __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (__attribute__((address_space(3))) void*)lds, 16, voffset, 0, 0, 0);
}
// The same with a wave-uniform byte offset in the scalar offset operand: a
// per-stage step added there costs no vector address arithmetic. NT: with the
// non-temporal hint (cache policy bit 1).
template <bool NT>
__device__ __forceinline__ void load_lds16_buf_so(__amdgpu_buffer_rsrc_t r, uint32_t voffset, uint32_t soffset,
                                                  bf16_t* lds) {
  __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (__attribute__((address_space(3))) void*)lds, 16, voffset, soffset, 0,
                                           NT ? 2 : 0);
}
// The same with the non-temporal hint (cache policy bit 1), for data read
// exactly once per call (decode weight streams).
__device__ __forceinline__ void load_lds16_buf_nt(__amdgpu_buffer_rsrc_t r, uint32_t voffset, bf16_t* lds) {
  __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (__attribute__((address_space(3))) void*)lds, 16, voffset, 0, 0, 2);
}
// Raw (stride 0) buffer resource over `bytes` bytes from `base`; loads past
// the end return zero.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t buffer_rsrc(const void* base, uint32_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), (short)0, (int)bytes, 0x00020000);
}

// s_waitcnt vmcnt(n) lgkmcnt(0): this wave's global->LDS fills older than
// its n most recent have landed, and its own LDS reads have returned.
template <int N>
__device__ __forceinline__ void wait_vmcnt_lgkm0() {
  static_assert(N >= 0 && N < 64, "vmcnt range");
  __builtin_amdgcn_s_waitcnt((N & 0xF) | ((N >> 4) << 14) | (0x7 << 4));
}

// Workgroup barrier without the release/acquire fences of __syncthreads():
// those wait for every outstanding global->LDS fill (vmcnt(0)) and would
// collapse a ring deeper than two stages. Callers wait explicitly first; the
// memory clobber keeps LDS accesses on their side of the barrier.
__device__ __forceinline__ void lds_barrier() { asm volatile("s_barrier" ::: "memory"); }

// The same barrier pinned in the instruction schedule: register-only work
// (MFMAs) may not move across it either.
__device__ __forceinline__ void lds_barrier_pinned() {
  __builtin_amdgcn_sched_barrier(0);
  asm volatile("s_barrier" ::: "memory");
  __builtin_amdgcn_sched_barrier(0);
}

// f(std::integral_constant<int, i>) for i = B .. E-1, unrolled at compile
// time (register arrays indexed by i stay in registers).
template <int B, int E, typename F>
__device__ __forceinline__ void static_for(F&& f) {
  if constexpr (B < E) {
    f(std::integral_constant<int, B>{});
    static_for<B + 1, E>(f);
  }
}

constexpr int min_c(int a, int b) { return a < b ? a : b; }

// ====================================================================== tile
// M > 64. Workgroup tile 64 QM x 64 QN, four waves (2 x 2, one per SIMD) of
// 32 QM x 32 QN, v_mfma_f32_32x32x16_bf16 with the accumulators (256 per lane
// at 256x256) in AGPRs. K runs in 64-wide stages through NS LDS slots filled
// by global->LDS DMA (buffer form); LDS rows are 128 B, their 16-byte chunks
// XOR-swizzled by (row / 2) % 8 so that the operand reads of 16 consecutive
// rows hit 16 distinct bank groups (the DMA lane addresses are chosen so
// that the linear fill lands swizzled).
//
// What bounds it. 256x256 (NS 2), many rounds: the MFMA rate at the clock the
// power cap allows. Between 65 and ~2000 rows 256x256 tiles leave most compute
// units idle (the 8B QKV GEMM at 256 rows: 24 workgroups, 82 us; as 128x64
// tiles 192 workgroups, 29 us) or end in a nearly empty round, and the smaller
// tiles are bound by the loads: with the MFMAs taken out, 256x128 at M 256,
// N 28672, K 4096 takes 64 of its 67 us, with the DMA taken out 47 us; 45 to
// 70 GB/s arrive per compute unit whatever the tile. So the smaller shapes
// keep as many stages in flight as LDS holds (128x128 at M 128, N 28672,
// K 4096: two slots 60 us, four 48, five 51).
//
// NT: for one tile row, where every weight is read by one workgroup only (and
// some launches of two rows, see launch_tile), the weights' loads carry the
// non-temporal hint and leave the caches to the activations, which all
// workgroups share (us, without -> with, weights cold): N 28672, K 4096 at 80
// rows 45.5 -> 41.5, at 256 61.8 -> 57.5; N 57344, K 8192 at 100 rows 160 ->
// 142, at 256 252 -> 221; N 10240, K 8192 at 128 rows 55 -> 53.
//
// Schedule of stage st (slot st % NS), four 16-k slices of QM QN MFMAs each.
// Every slice interleaves with its MFMAs:
//  * the reads of the next slice's QM + QN fragments, spread from the first
//    MFMA on, in the order the next slice first uses them (a0 b0 b1 .. a1 a2
//    ..), so its MFMAs wait only for their own;
//  * DMA instructions, one after every other MFMA from the second where the
//    slice is long enough, else evenly: in slice 3 the first part of stage
//    st+NS into slot st % NS, in slices 0 to 2 the rest of stage st+NS-1.
// After slice 2: wait for stage st+1 and this stage's reads, one barrier
// (slot st % NS is free from there, and slice 3 reads stage st+1's first
// fragments). Issued in bursts, DMA or reads back up the address unit and
// the LDS queue and stall the waves' instruction streams. With two slots the
// 16 DMA instructions of 256x256 go 7 / 7 / 2 over slices 3, 0, 1: loads
// issued in slice 1 have only a slice and a half to land before that wait,
// which an L2 miss outlasts (6 / 5 / 5 was 2% slower on the gate_up shape).
// The last stages run in a loop with the slot computed: unrolled per
// remainder, the 256x256 form spilled 2000 registers.
namespace tile {
constexpr int BK = 64, NT = 256;
constexpr int CPR = BK / 8, RPL = 64 / CPR;  // 8 chunks per row, 8 rows per DMA instruction
__device__ __forceinline__ int swz(int row, int ch) { return row * BK + ((ch ^ ((row >> 1) & 7)) << 3); }
template <int QM, int QN, int NS>
struct Geo {
  static constexpr int BM = 64 * QM, BN = 64 * QN;                // 2 x 2 waves of 32 QM x 32 QN
  static constexpr int A_ELTS = BM * BK, STAGE = (BM + BN) * BK;  // bf16 elements
  static constexpr int A_LOADS = BM / RPL / 4, B_LOADS = BN / RPL / 4, LOADS = A_LOADS + B_LOADS;  // per wave
  static constexpr int MF = QM * QN, RD = QM + QN;                // MFMAs and fragment reads per slice
  // DMA split over slices 3 (of the stage before), 0, 1, 2
  static constexpr int D3 = NS == 2 ? (LOADS == 16 ? 7 : LOADS / 2) : (LOADS + 3) / 4;
  static constexpr int D0 = NS == 2 ? (LOADS == 16 ? 7 : LOADS - D3) : (LOADS - D3 + 2) / 3;
  static constexpr int D1 = NS == 2 ? LOADS - D3 - D0 : (LOADS - D3 - D0 + 1) / 2;
  static constexpr int D2 = LOADS - D3 - D0 - D1;
  static constexpr int ROWF = 32 * QN + 8;  // staged output row: the two lane halves, 4 rows apart, land 32 banks apart
  static constexpr size_t RING = (size_t)NS * STAGE * 2, STAGING = (size_t)4 * 32 * ROWF * 4;
  // A ring of more than half the LDS leaves one workgroup per compute unit.
  // Such a launch takes all 160 KiB, so that no other stream's workgroup
  // shares the unit either: beside the decode attention of a mixed step (4 x
  // 512 chunk rows + 32 long contexts) the shapes that leave it room run the
  // step in 1313 us, shut out it takes 1154 us.
  static constexpr size_t LDS_BYTES = RING > 80 * 1024 ? 160 * 1024 : RING > STAGING ? RING : STAGING;
  static_assert(RING <= 160 * 1024 && STAGING <= 160 * 1024, "LDS per workgroup");
};
// items [lo, hi) of `n` that go after MFMA q of `mf`
constexpr int share(int n, int mf, int q) { return n * q / mf; }
}  // namespace tile

template <int QM, int QN, int NS, bool NT, int EPI, typename TR, typename TC>
__global__ __launch_bounds__(256) void gemm_tile_kernel(const bf16_t* __restrict__ A, const bf16_t* __restrict__ W,
                                                        const TR* __restrict__ R, TC* __restrict__ C, int M, int N,
                                                        int K, int tiles_n, int group, int splits) {
  using namespace tile;
  using G = Geo<QM, QN, NS>;
  constexpr int BM = G::BM, BN = G::BN, STAGE = G::STAGE, A_LOADS = G::A_LOADS, B_LOADS = G::B_LOADS, LOADS = G::LOADS;
  constexpr int MF = G::MF, RD = G::RD;
  extern __shared__ __attribute__((aligned(16))) bf16_t smem[];

  // XCD-aware tile order: consecutive workgroup ids go round-robin over the
  // 8 XCDs; give each XCD a contiguous range of tiles, walked in groups of
  // `group` tile-rows across N, so that tiles sharing A and W panels meet in
  // the same L2.
  // With splits > 1 (EPI 0, fp32 C) the grid holds every tile once per K
  // split, split-major: split s covers stages [s T / splits, (s + 1) T /
  // splits) and stores its partial at C + s M N.
  const int nwg = gridDim.x;
  int id = blockIdx.x;
  {
    const int x = id & 7, per = nwg >> 3, rem = nwg & 7;
    id = x * per + min(x, rem) + (id >> 3);
  }
  const int n_tiles = nwg / splits;
  const int ks = id / n_tiles;
  id -= ks * n_tiles;
  const int tiles_m = n_tiles / tiles_n;
  const int group_sz = group * tiles_n;
  const int first_m = (id / group_sz) * group;
  const int gm = min(group, tiles_m - first_m);
  const int tm = first_m + (id % group_sz) % gm;
  const int tn = (id % group_sz) / gm;
  const int m0 = tm * BM, n0 = tn * BN;

  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int wm = wave >> 1, wn = wave & 1;
  // DMA sources: buffer resources at the tile's A rows and W blocks, 32-bit
  // lane byte offsets (rows past M read row M-1, results unused)
  const int lrow = lane / CPR, lpos = lane % CPR;
  uint32_t aoff[A_LOADS], boff[B_LOADS];
#pragma unroll
  for (int i = 0; i < A_LOADS; ++i) {
    const int row = (wave * A_LOADS + i) * RPL + lrow;
    aoff[i] = ((uint32_t)(min(m0 + row, M - 1) - m0) * K + (lpos ^ ((row >> 1) & 7)) * 8) * 2;
  }
#pragma unroll
  for (int i = 0; i < B_LOADS; ++i) {  // tiled W: rows of 64-row block row/64, k-tile added per stage
    const int row = (wave * B_LOADS + i) * RPL + lrow;
    boff[i] = ((uint32_t)(row >> 6) * (K / 64) * kWTileElts + (row & 63) * 64 + (lpos ^ ((row >> 1) & 7)) * 8) * 2;
  }
  static_assert(BK == kWTile, "one W tile per stage");
  const __amdgpu_buffer_rsrc_t rA = buffer_rsrc(A + (long)m0 * K, (uint32_t)min(M - m0, BM) * K * 2);
  const __amdgpu_buffer_rsrc_t rW =
      buffer_rsrc(W + (long)(n0 >> 6) * (K / 64) * kWTileElts, (uint32_t)(BN / 64) * (K / 64) * kWTileElts * 2);
  const int T_all = K / BK;
  const int st0 = ks * T_all / splits, T = (ks + 1) * T_all / splits - st0;  // this workgroup's stages
  // DMA instruction l (0..LOADS-1) of stage s into slot dslot (= s % NS);
  // the stage's step rides in the scalar offset
  auto dma = [&](int s, int dslot, int l) __attribute__((always_inline)) {
    bf16_t* st = smem + dslot * STAGE;
    if (l < A_LOADS)
      load_lds16_buf_so<false>(rA, aoff[l], (s + st0) * BK * 2, st + (wave * A_LOADS + l) * RPL * BK);
    else
      load_lds16_buf_so<NT>(rW, boff[l - A_LOADS], (s + st0) * kWTileElts * 2,
                            st + G::A_ELTS + (wave * B_LOADS + l - A_LOADS) * RPL * BK);
  };

  // 32x32x16 operands: lane (h, r) holds row r of a 32-row block, k 8h..8h+7
  // of a 16-k slice; fragments double-buffered by slice parity
  const int h = lane >> 5, r32 = lane & 31;
  bf16x8_t fa[2][QM], fb[2][QN];
  // fragment r (0..QM+QN-1) of slice sl, in first-use order: a0 b0 .. b(QN-1) a1 .. a(QM-1)
  auto read_frag = [&](int slot, int sl, int r) __attribute__((always_inline)) {
    const bf16_t* a = smem + slot * STAGE;
    if (r == 0)
      fa[sl & 1][0] = __builtin_bit_cast(bf16x8_t, *(const uint4*)(a + swz(wm * 32 * QM + r32, 2 * sl + h)));
    else if (r <= QN)
      fb[sl & 1][r - 1] = __builtin_bit_cast(
          bf16x8_t, *(const uint4*)(a + G::A_ELTS + swz(wn * 32 * QN + (r - 1) * 32 + r32, 2 * sl + h)));
    else
      fa[sl & 1][r - QN] =
          __builtin_bit_cast(bf16x8_t, *(const uint4*)(a + swz(wm * 32 * QM + (r - QN) * 32 + r32, 2 * sl + h)));
  };
  f32x16_t acc[QM][QN];
#pragma unroll
  for (int i = 0; i < QM; ++i)
#pragma unroll
    for (int j = 0; j < QN; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;
  // an (empty) AGPR operand makes the compiler select the AGPR form of the
  // MFMAs, which keeps the accumulators in place in the AGPR file
  asm volatile("" ::"a"(0.f));
  auto mfma = [&](int sl, int q) __attribute__((always_inline)) {
    acc[q / QN][q % QN] =
        __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[sl & 1][q / QN], fb[sl & 1][q % QN], acc[q / QN][q % QN], 0, 0, 0);
  };

  // stage st, in LDS slot st % NS. `slotc`: that slot as an integral constant
  // where the caller knows it (LDS addresses then fold into instruction
  // offsets) and st + NS < T holds (FULL: nothing below is conditional);
  // else an int.
  auto stage = [&](int st, auto slotc) __attribute__((always_inline)) {
    constexpr bool FULL = !std::is_same<decltype(slotc), int>::value;
    const int slot = slotc, nslot = FULL ? (slot + 1) % NS : (slot + 1 == NS ? 0 : slot + 1),
              pslot = FULL ? (slot + NS - 1) % NS : (slot == 0 ? NS - 1 : slot - 1);
    const bool more = FULL || st + 1 < T;                         // a stage follows
    const bool far = FULL || st + NS < T;                         // first part of stage st+NS
    const bool next = st > 0 && (FULL || st + NS - 1 < T);        // rest of stage st+NS-1 (0..NS-1 come whole with the prologue)
    auto slice = [&](auto slc) __attribute__((always_inline)) {
      constexpr int sl = decltype(slc)::value;
      constexpr int DN = sl == 0 ? G::D0 : sl == 1 ? G::D1 : sl == 2 ? G::D2 : G::D3;
      constexpr int DB = sl == 0 ? G::D3 : sl == 1 ? G::D3 + G::D0 : sl == 2 ? G::D3 + G::D0 + G::D1 : 0;
      // instruction d of the slice's DN goes after MFMA 1 + 2 d where the slice has that many, else evenly
      constexpr bool every2 = 1 + 2 * (DN - 1) < MF;
      const int rslot = sl == 3 ? nslot : slot;
      const bool rd = sl < 3 || more;
      const bool dd = sl == 3 ? far : next;
      const int ds = sl == 3 ? st + NS : st + NS - 1;
      static_for<0, MF>([&](auto qc) __attribute__((always_inline)) {
        constexpr int q = decltype(qc)::value;
        mfma(sl, q);
        constexpr int r0 = RD <= MF ? min_c(q, RD) : share(RD, MF, q), r1 = RD <= MF ? min_c(q + 1, RD) : share(RD, MF, q + 1);
        constexpr int d0 = every2 ? min_c(q / 2, DN) : share(DN, MF, q), d1 = every2 ? min_c((q + 1) / 2, DN) : share(DN, MF, q + 1);
        if (rd) static_for<r0, r1>([&](auto rc) __attribute__((always_inline)) { read_frag(rslot, (sl + 1) & 3, decltype(rc)::value); });
        if (dd) static_for<d0, d1>([&](auto dc) __attribute__((always_inline)) {
          dma(ds, sl == 3 ? slot : pslot, DB + decltype(dc)::value);
        });
      });
      if constexpr (FULL) {
        static_for<0, MF>([&](auto qc) __attribute__((always_inline)) {
          constexpr int q = decltype(qc)::value;
          constexpr int rn = RD <= MF ? min_c(q + 1, RD) - min_c(q, RD) : share(RD, MF, q + 1) - share(RD, MF, q);
          constexpr int dn = every2 ? min_c((q + 1) / 2, DN) - min_c(q / 2, DN) : share(DN, MF, q + 1) - share(DN, MF, q);
          __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);                    // MFMA
          if constexpr (rn > 0) __builtin_amdgcn_sched_group_barrier(0x100, rn, 0);  // LDS read
          if constexpr (dn > 0) __builtin_amdgcn_sched_group_barrier(0x020, dn, 0);  // VMEM read (DMA)
        });
      }
      if constexpr (sl == 2) {
        __builtin_amdgcn_sched_barrier(0);
        // stage st+1 landed (the NS - 2 stages after it, as far as there are
        // any, may be in flight), this stage's reads returned
        if constexpr (FULL) {
          wait_vmcnt_lgkm0<(NS - 2) * LOADS>();
          lds_barrier_pinned();
        } else if (more) {
          const int after = min(T - 2 - st, NS - 2);
          static_for<0, NS - 1>([&](auto ac) __attribute__((always_inline)) {
            if (after == decltype(ac)::value) wait_vmcnt_lgkm0<decltype(ac)::value * LOADS>();
          });
          lds_barrier_pinned();
        }
      }
    };
    slice(std::integral_constant<int, 0>{});
    slice(std::integral_constant<int, 1>{});
    slice(std::integral_constant<int, 2>{});
    slice(std::integral_constant<int, 3>{});
  };

  // prologue: stages 0 .. NS-1 whole, stage 0 landed everywhere, its first
  // fragments read
  static_for<0, NS>([&](auto sc) __attribute__((always_inline)) {
    constexpr int s = decltype(sc)::value;
    if (s < T) {
#pragma unroll
      for (int l = 0; l < LOADS; ++l) dma(s, s, l);
    }
  });
  if (T >= NS) wait_vmcnt_lgkm0<(NS - 1) * LOADS>();
  else wait_vmcnt_lgkm0<0>();
  lds_barrier_pinned();
#pragma unroll
  for (int r = 0; r < RD; ++r) read_frag(0, 0, r);
  int st = 0;
  for (; st + 2 * NS - 1 < T; st += NS)  // NS stages per trip: every slot known at compile time
    static_for<0, NS>([&](auto sc) __attribute__((always_inline)) { stage(st + decltype(sc)::value, sc); });
  for (int slot = 0; st < T; ++st) {  // st is a multiple of NS here
    stage(st, slot);
    if (++slot == NS) slot = 0;
  }

  // epilogue: acc[i][j][r] is C[32 i + 8 (r / 4) + 4 h + r % 4][32 j + r32]
  // of the wave tile. Each 32-row block goes through a wave-private LDS
  // staging area (fp32, rows padded by 8 floats: the two lane halves,
  // 4 rows apart, land 32 banks apart), then every lane reads V consecutive
  // columns and the global stores (and residual loads) are 16 bytes per
  // lane: a few wide VMEM instructions instead of one per (row group,
  // column block). SwiGLU: the wave's column blocks alternate gate and up
  // (the 32-row interleave of w_gate_up), block 2p pairs with 2p + 1.
  constexpr int ROWF = G::ROWF, WT = 32 * QN;
  const int rbase = m0 + wm * 32 * QM, cbase = n0 + wn * WT;
  constexpr int V = std::is_same<TC, bf16_t>::value ? 8 : 4;  // columns per lane
  constexpr int OUT_COLS = EPI == 2 ? WT / 2 : WT;
  constexpr int LPR = OUT_COLS / V, RPP = 64 / LPR;  // lanes per row, rows per pass
  const long ldc = EPI == 2 ? N / 2 : N;
  const long ccol = EPI == 2 ? cbase / 2 : cbase;
  C += (long)ks * M * ldc;  // this split's partial
  constexpr int NPASS = 32 / RPP;
  // residual operand of one pass: V values of row `row` from column `oc`
  using RRaw = typename std::conditional<std::is_same<TR, float>::value, float4,
                                         typename std::conditional<V == 8, uint4, uint2>::type>::type;
  constexpr int RCH = std::is_same<TR, float>::value ? V / 4 : 1;  // RRaw loads per pass
  // Residual loads run one 32-row block ahead of the block being stored
  // (two register sets), the first block's issued before the staging
  // barrier, so that the HBM latency of the loads, which every CU issues at
  // about the same moment, is exposed once per tile instead of once per
  // block. Block i + 1's rows are disjoint from block i's, so the loads may
  // precede block i's stores even where R aliases C, and every element is
  // still read before it is written.
  RRaw rr[2][EPI == 1 ? NPASS : 1][RCH];
  auto load_r = [&](int i) __attribute__((always_inline)) {
    if constexpr (EPI == 1) {
#pragma unroll
      for (int pass = 0; pass < NPASS; ++pass) {
        const int row = rbase + i * 32 + pass * RPP + lane / LPR, oc = (lane % LPR) * V;
        const long idx = (long)min(row, M - 1) * ldc + ccol + oc;  // rows past M: a valid row, result unused
#pragma unroll
        for (int q = 0; q < RCH; ++q) rr[i & 1][pass][q] = *(const RRaw*)(R + idx + q * 4);
      }
    }
  };
  load_r(0);
  lds_barrier_pinned();  // every wave is done reading operand slots
  float* stg = (float*)smem + wave * (32 * ROWF);
#pragma unroll
  for (int i = 0; i < QM; ++i) {
    if (i + 1 < QM) load_r(i + 1);
#pragma unroll
    for (int j = 0; j < QN; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) stg[(8 * (r >> 2) + 4 * h + (r & 3)) * ROWF + j * 32 + r32] = acc[i][j][r];
    // LDS accesses of one wave complete in order: the reads below see the writes
#pragma unroll
    for (int pass = 0; pass < NPASS; ++pass) {
      const int lr = pass * RPP + lane / LPR, oc = (lane % LPR) * V;
      const int row = rbase + i * 32 + lr;
      float v[V];
      if constexpr (EPI == 2) {
        const int p = oc / 32, c = oc % 32;
        const float* g = stg + lr * ROWF + p * 64 + c;
#pragma unroll
        for (int e = 0; e < V; e += 4) {
          const float4 gv = *(const float4*)(g + e), uv = *(const float4*)(g + 32 + e);
          v[e] = silu_fast(gv.x) * uv.x;
          v[e + 1] = silu_fast(gv.y) * uv.y;
          v[e + 2] = silu_fast(gv.z) * uv.z;
          v[e + 3] = silu_fast(gv.w) * uv.w;
        }
      } else {
#pragma unroll
        for (int e = 0; e < V; e += 4) {
          const float4 a4 = *(const float4*)(stg + lr * ROWF + oc + e);
          v[e] = a4.x;
          v[e + 1] = a4.y;
          v[e + 2] = a4.z;
          v[e + 3] = a4.w;
        }
      }
      if constexpr (EPI == 1) {
        if constexpr (std::is_same<TR, float>::value) {
#pragma unroll
          for (int q = 0; q < RCH; ++q) {
            v[4 * q] += rr[i & 1][pass][q].x;
            v[4 * q + 1] += rr[i & 1][pass][q].y;
            v[4 * q + 2] += rr[i & 1][pass][q].z;
            v[4 * q + 3] += rr[i & 1][pass][q].w;
          }
        } else if constexpr (V == 8) {
          const uint32_t w4[4] = {rr[i & 1][pass][0].x, rr[i & 1][pass][0].y, rr[i & 1][pass][0].z, rr[i & 1][pass][0].w};
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            v[2 * e] += bf_lo(w4[e]);
            v[2 * e + 1] += bf_hi(w4[e]);
          }
        } else {
          v[0] += bf_lo(rr[i & 1][pass][0].x);
          v[1] += bf_hi(rr[i & 1][pass][0].x);
          v[2] += bf_lo(rr[i & 1][pass][0].y);
          v[3] += bf_hi(rr[i & 1][pass][0].y);
        }
      }
      if (row >= M) continue;
      const long idx = (long)row * ldc + ccol + oc;
      if constexpr (std::is_same<TC, bf16_t>::value) {
        typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
        __builtin_nontemporal_store(u32x4{pack_bf2(v[0], v[1]), pack_bf2(v[2], v[3]), pack_bf2(v[4], v[5]),
                                          pack_bf2(v[6], v[7])}, (u32x4*)(C + idx));
      } else {
        typedef float f32x4 __attribute__((ext_vector_type(4)));
        __builtin_nontemporal_store(f32x4{v[0], v[1], v[2], v[3]}, (f32x4*)(C + idx));
      }
    }
  }
}

// `cols` of the N output columns: W, R and C point at the first of them.
template <int QM, int QN, int NS, bool NT, int EPI, typename TR, typename TC>
int launch_tile_g(int M, int N, int cols, int K, const void* A, const void* W, const void* R, void* C, hipStream_t st,
                  int splits, int group) {
  using G = tile::Geo<QM, QN, NS>;
  static const hipError_t attr = hipFuncSetAttribute((const void*)gemm_tile_kernel<QM, QN, NS, NT, EPI, TR, TC>,
                                                     hipFuncAttributeMaxDynamicSharedMemorySize, (int)G::LDS_BYTES);
  if (attr != hipSuccess) return -1;
  const int tiles_m = (M + G::BM - 1) / G::BM, tiles_n = cols / G::BN;
  hipLaunchKernelGGL((gemm_tile_kernel<QM, QN, NS, NT, EPI, TR, TC>), dim3(tiles_m * tiles_n * splits), dim3(tile::NT),
                     G::LDS_BYTES, st, (const bf16_t*)A, (const bf16_t*)W, (const TR*)R, (TC*)C, M, N, K, tiles_n,
                     group, splits);
  return 0;
}

// Every instance the launcher reaches, X(QM, QN, NS, NT, EPI, TR, TC), by the
// source file that compiles it. NS: ring slots that fit 160 KiB of LDS.
#define PS_TILE_INSTANCES_NT(X, QM, QN, NS, NT)                                                               \
  X(QM, QN, NS, NT, 0, float, bf16_t) X(QM, QN, NS, NT, 0, float, float) X(QM, QN, NS, NT, 1, bf16_t, float)  \
  X(QM, QN, NS, NT, 1, float, bf16_t)
#define PS_TILE_INSTANCES_ALL(X, QM, QN, NS) \
  PS_TILE_INSTANCES_NT(X, QM, QN, NS, false) PS_TILE_INSTANCES_NT(X, QM, QN, NS, true)
#define PS_TILE_INSTANCES_SWIGLU(X, QM, QN, NS) \
  X(QM, QN, NS, false, 2, float, bf16_t) X(QM, QN, NS, true, 2, float, bf16_t)
#define PS_TILE_INSTANCES_256(X)                                                   \
  PS_TILE_INSTANCES_ALL(X, 4, 4, 2) PS_TILE_INSTANCES_SWIGLU(X, 4, 4, 2)           \
  X(4, 4, 2, false, 1, bf16_t, bf16_t) X(4, 4, 2, false, 1, float, float) X(4, 4, 2, false, 2, float, float)
#define PS_TILE_INSTANCES_WIDE(X)                                                  \
  PS_TILE_INSTANCES_ALL(X, 3, 4, 2) PS_TILE_INSTANCES_SWIGLU(X, 3, 4, 2)           \
  PS_TILE_INSTANCES_ALL(X, 2, 4, 3) PS_TILE_INSTANCES_SWIGLU(X, 2, 4, 3)
#define PS_TILE_INSTANCES_TALL(X)                                                  \
  PS_TILE_INSTANCES_ALL(X, 4, 2, 3) PS_TILE_INSTANCES_SWIGLU(X, 4, 2, 3)           \
  PS_TILE_INSTANCES_ALL(X, 3, 2, 3) PS_TILE_INSTANCES_SWIGLU(X, 3, 2, 3)
#define PS_TILE_INSTANCES_SMALL(X)                                                 \
  PS_TILE_INSTANCES_ALL(X, 2, 2, 4) PS_TILE_INSTANCES_SWIGLU(X, 2, 2, 4)           \
  PS_TILE_INSTANCES_ALL(X, 2, 1, 6) PS_TILE_INSTANCES_NT(X, 1, 1, 5, false)
#define PS_TILE_INSTANCES(X) \
  PS_TILE_INSTANCES_256(X) PS_TILE_INSTANCES_WIDE(X) PS_TILE_INSTANCES_TALL(X) PS_TILE_INSTANCES_SMALL(X)
#define PS_TILE_INSTANTIATE(QM, QN, NS, NT, EPI, TR, TC)                                                        \
  template int launch_tile_g<QM, QN, NS, NT, EPI, TR, TC>(int, int, int, int, const void*, const void*,         \
                                                          const void*, void*, hipStream_t, int, int);

}  // namespace ps
