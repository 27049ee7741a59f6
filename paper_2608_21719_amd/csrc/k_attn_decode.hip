// Decode attention over the paged KV cache (gfx950).
//
// Split-K: a work item is (batch entry, logical page range, kv head). Its
// four waves walk the range's 16-token pages in logical order (wave w takes
// pages w, w+4, ...), so the arithmetic never depends on where pages sit
// physically. Per page a wave reads the 4 KiB key block with 16-byte loads
// and the 4 KiB V^T block with 8-byte loads, non-temporal (KV is streamed
// once per step), keeping kPrefetch pages in flight beyond the one it works
// on; the block table is read with scalar loads, so fetching the next page
// id never waits on the vector loads already in flight. The kv head is the
// fastest grid index: workgroups running together read the adjacent heads
// of the same pages. A launch may cap its workgroups (the mixed step does,
// to leave compute units to the GEMMs beside it); each then walks items
// y, y + gridDim.y, ... in turn. Each page does all of the group's query heads at once
// on the matrix cores:
//
//   S^T[tok, head] = K[tok, :] . q[head, :]     4 x v_mfma_f32_16x16x32_bf16
//   O[head, dim]  += P[head, tok] V[tok, dim]   8 x v_mfma_f32_16x16x16_bf16
//
// The 16-row MFMA tile holds the G (<= 16) heads of one KV group; rows
// beyond G are padding. The S^T output layout (lane = head, 4 tokens per
// lane) is exactly the A-operand layout P needs, so no shuffle sits between
// the two products. Online softmax runs in base 2 on fp32 scores; P is
// rounded to bf16 for the PV product and the normaliser sums those same
// rounded values (so V == 1 gives exactly 1). The pass is bound by HBM:
// 4 FLOP per KV byte.
//
// A second kernel merges the splits of each (sequence, head) in split order
// (log-sum-exp), which keeps the result deterministic; a sequence in one split
// is finished by the attention kernel itself.
#include "common.h"
#include "launch.h"

#include <type_traits>

namespace ps {

constexpr int kHd = 128;      // head_dim of the MFMA path
constexpr int kPrefetch = 2;  // pages in flight per wave beyond the current one

typedef uint32_t u32x2_t __attribute__((ext_vector_type(2)));

// ROPE: the launch also does RoPE and the KV write of the step's new tokens (a
// launch of its own takes 4.7 to 8.6 us; taken where one round of workgroups
// does the batch). Every workgroup rotates its own G query heads from the QKV
// projection while its first pages are on their way; the one whose range ends
// with the sequence's last page also rotates the new key, writes key and value
// to the page, and puts them into its own copy of that page in registers, so
// no read depends on the write. The arithmetic is rope_kvwrite_kernel's.
template <int G, bool ROPE>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2))) void decode_attn_kernel(
    const bf16_t* __restrict__ q, bf16_t* __restrict__ pool, const SeqInfo* __restrict__ si,
    const int32_t* __restrict__ bt, const DecodeItem* __restrict__ items, float* __restrict__ part_o,
    float* __restrict__ part_ml, bf16_t* __restrict__ out, int n_kv, int n_items, float scale_log2, DecodeRope rp) {
  static_assert(G <= 16, "one 16-row MFMA tile per KV group");
  __shared__ __attribute__((aligned(16))) bf16_t s_q[ROPE ? G * kHd : 8], s_k[ROPE ? kHd : 8], s_v[ROPE ? kHd : 8];
  constexpr int D = kPrefetch;
  const int kvh = blockIdx.x;
  // items blockIdx.y, + gridDim.y, ...: one each when the grid covers them
  // all, several when the launch caps its workgroups
  for (int iy = blockIdx.y; iy < n_items; iy += gridDim.y) {
  const DecodeItem it = items[iy];
  const SeqInfo s = si[it.b];
  const int kv_len = s.kv_before + s.n_new;
  const int n_q = n_kv * G;
  // wave index made wave-uniform so page ids and page addresses stay scalar
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  const int g = lane >> 4, c = lane & 15;

  const int last_page = (kv_len - 1) / kPageTokens;
  const bool has_new = ROPE && it.page_end == last_page + 1;  // this range holds the new token
  // QKV inputs of this workgroup: (x1, x2) of pair j of a head per thread
  constexpr int QP = ROPE ? (G * (kHd / 2) + 255) / 256 : 1;  // query pairs per thread
  float qx[QP][2] = {}, kx[2] = {}, vx = 0.f;
  double ang = 0.0;
  if constexpr (ROPE) {
    const long row = (long)it.b * (n_q + 2 * n_kv) * kHd;
    const int t = threadIdx.x, j = t & 63;
    ang = (double)s.kv_before * rp.inv_freq[j];
    auto load = [&](auto get) __attribute__((always_inline)) {
#pragma unroll
      for (int u = 0; u < QP; ++u) {
        const int head = (t >> 6) + 4 * u;
        if (head < G) {
          const long col = row + (long)(kvh * G + head) * kHd + j;
          qx[u][0] = get(col);
          qx[u][1] = get(col + kHd / 2);
        }
      }
      if (has_new) {
        if (t < 64) {
          const long col = row + (long)(n_q + kvh) * kHd + j;
          kx[0] = get(col);
          kx[1] = get(col + kHd / 2);
        } else if (t < 64 + kHd) {
          vx = get(row + (long)(n_q + n_kv + kvh) * kHd + t - 64);
        }
      }
    };
    auto sum = [&](auto sc) __attribute__((always_inline)) {
      load([&](long col) __attribute__((always_inline)) {
        constexpr int S = decltype(sc)::value;
        float p[S];
#pragma unroll
        for (int i = 0; i < S; ++i) p[i] = rp.part[i * rp.mn + col];
        float a = 0.f;
#pragma unroll
        for (int i = 0; i < S; ++i) a += p[i];
        return bf2f(f2bf(a));
      });
    };
    switch (rp.splits) {
      case 2: sum(std::integral_constant<int, 2>{}); break;
      case 3: sum(std::integral_constant<int, 3>{}); break;
      case 4: sum(std::integral_constant<int, 4>{}); break;
      case 8: sum(std::integral_constant<int, 8>{}); break;
      default: load([&](long col) __attribute__((always_inline)) { return bf2f(rp.qkv[col]); }); break;
    }
  }

  // Q operand (B of the S^T product): lane holds q[head c][32j + 8g .. +8].
  bf16x8_t qb[4];
  if constexpr (!ROPE) {
    const bf16_t* qp = q + ((long)it.b * n_q + kvh * G + (c < G ? c : 0)) * kHd + 8 * g;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      uint4 w = (c < G) ? *(const uint4*)(qp + 32 * j) : make_uint4(0, 0, 0, 0);
      qb[j] = __builtin_bit_cast(bf16x8_t, w);
    }
  }

  float m = -INFINITY, l = 0.f;
  f32x4_t acc[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) acc[i] = f32x4_t{0.f, 0.f, 0.f, 0.f};

  const int32_t* btr = bt + s.bt_off;
  const int koff = c * kHd + 8 * g;                               // + 32 j
  const int voff = kPageTokens * kHd + c * kPageTokens + 4 * g;   // + 16 blk kPageTokens
  const long head_off = (long)kvh * (2L * kPageTokens * kHd);
  const long page_stride = (long)n_kv * (2L * kPageTokens * kHd);

  // three static register sets form the page ring (two pages in flight while
  // one is consumed); a ring indexed at run time would be copied through
  // registers, and each copy of an in-flight load waits for it
  static_assert(kPrefetch == 2, "the page ring below is unrolled for two pages in flight");
  struct PageRegs {
    uint4 k[4];
    uint2 v[8];
  };
  PageRegs r0, r1, r2;
  auto load_page = [&](int p, PageRegs& r) {
    const bf16_t* base = pool + (long)btr[p] * page_stride + head_off;
#pragma unroll
    for (int j = 0; j < 4; ++j)
      r.k[j] = __builtin_bit_cast(uint4, __builtin_nontemporal_load((const u32x4_t*)(base + koff + 32 * j)));
#pragma unroll
    for (int blk = 0; blk < 8; ++blk)
      r.v[blk] = __builtin_bit_cast(
          uint2, __builtin_nontemporal_load((const u32x2_t*)(base + voff + 16 * blk * kPageTokens)));
  };

  // consume one page held in `cur`; `tailc`: it may be the sequence's last
  auto page_compute = [&](int p, PageRegs& cur, auto tailc) {
    if constexpr (ROPE && decltype(tailc)::value) {
      if (p == last_page) {  // the new token's slot: its key and value from LDS
        const int slot = (kv_len - 1) % kPageTokens;
        if (c == slot) {
#pragma unroll
          for (int j = 0; j < 4; ++j) cur.k[j] = *(const uint4*)(s_k + 32 * j + 8 * g);
        }
        if (g == slot >> 2) {
          const uint32_t keep = (slot & 1) ? 0x0000ffffu : 0xffff0000u;
#pragma unroll
          for (int blk = 0; blk < 8; ++blk) {
            const uint32_t v = (uint32_t)s_v[16 * blk + c] << ((slot & 1) * 16);
            if (slot & 2) cur.v[blk].y = (cur.v[blk].y & keep) | v;
            else cur.v[blk].x = (cur.v[blk].x & keep) | v;
          }
        }
      }
    }
    // tokens past the written length (last page only) hold stale memory:
    // zero their V so 0 * garbage cannot produce NaN (branch-free, so no
    // wait on the page's loads is placed on a path of its own)
    const int valid = (p == last_page) ? kv_len - p * kPageTokens : kPageTokens;  // 1..16
    const uint32_t m0 = (4 * g + 0 < valid ? 0x0000ffffu : 0u) | (4 * g + 1 < valid ? 0xffff0000u : 0u);
    const uint32_t m1 = (4 * g + 2 < valid ? 0x0000ffffu : 0u) | (4 * g + 3 < valid ? 0xffff0000u : 0u);
#pragma unroll
    for (int blk = 0; blk < 8; ++blk) cur.v[blk] = make_uint2(cur.v[blk].x & m0, cur.v[blk].y & m1);

    f32x4_t st = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int j = 0; j < 4; ++j)
      st = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, cur.k[j]), qb[j], st, 0, 0, 0);
    // st[r] = score(token 4g + r, head c)
    float sc[4];
    float mx = -INFINITY;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int tok = p * kPageTokens + 4 * g + r;
      sc[r] = (tok < kv_len) ? st[r] * scale_log2 : -INFINITY;
      mx = fmaxf(mx, sc[r]);
    }
    mx = fmaxf(mx, __shfl_xor(mx, 16));
    mx = fmaxf(mx, __shfl_xor(mx, 32));
    const float m_new = fmaxf(m, mx);
    const float base = m_new == -INFINITY ? 0.f : m_new;  // only scores of -inf yet: their weights are 0, not NaN
    const float alpha = exp2f(m - base);
    float pr[4];
    uint32_t pk[2];
#pragma unroll
    for (int r = 0; r < 2; ++r) {
      pk[r] = pack_bf2(exp2f(sc[2 * r] - base), exp2f(sc[2 * r + 1] - base));
      pr[2 * r] = bf_lo(pk[r]);
      pr[2 * r + 1] = bf_hi(pk[r]);
    }
    l = l * alpha + (pr[0] + pr[1] + pr[2] + pr[3]);
    m = m_new;
    // acc rows are heads 4g + r: fetch their rescale factors
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const float a_r = __shfl(alpha, 4 * g + r);
#pragma unroll
      for (int blk = 0; blk < 8; ++blk) acc[blk][r] *= a_r;
    }
    const s16x4_t pa = __builtin_bit_cast(s16x4_t, make_uint2(pk[0], pk[1]));
#pragma unroll
    for (int blk = 0; blk < 8; ++blk)
      acc[blk] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(pa, __builtin_bit_cast(s16x4_t, cur.v[blk]), acc[blk],
                                                           0, 0, 0);
  };

  // wave pages p0, p0 + 4, ...: r0 holds page p and r1 page p + 4 at the top
  // of every round; a round consumes three pages and requests three
  const int end = it.page_end;
  int p = it.page_begin + wave;
  if (p < end) load_page(p, r0);
  __builtin_amdgcn_sched_barrier(0);  // page p's loads first (the wait for it below counts on that order)
  if (p + 4 < end) load_page(p + 4, r1);
  __builtin_amdgcn_sched_barrier(0);
  if constexpr (ROPE) {
    const int t = threadIdx.x, j = t & 63;
    double sd, cd;
    sincos(ang, &sd, &cd);
    const float cs = (float)cd, sn = (float)sd;
    float y1, y2;
#pragma unroll
    for (int u = 0; u < QP; ++u) {
      const int head = (t >> 6) + 4 * u;
      if (head < G) {
        rope_pair(qx[u][0], qx[u][1], cs, sn, y1, y2);
        s_q[head * kHd + j] = f2bf(y1);
        s_q[head * kHd + j + kHd / 2] = f2bf(y2);
      }
    }
    if (has_new) {
      bf16_t* pg = pool + (long)btr[last_page] * page_stride + head_off;
      const int slot = (kv_len - 1) % kPageTokens;
      if (t < 64) {
        rope_pair(kx[0], kx[1], cs, sn, y1, y2);
        const bf16_t k1 = f2bf(y1), k2 = f2bf(y2);
        s_k[j] = k1;
        s_k[j + kHd / 2] = k2;
        pg[slot * kHd + j] = k1;
        pg[slot * kHd + j + kHd / 2] = k2;
      } else if (t < 64 + kHd) {
        const bf16_t v = f2bf(vx);
        s_v[t - 64] = v;
        pg[kPageTokens * kHd + (t - 64) * kPageTokens + slot] = v;
      }
    }
    // LDS only: a full fence would wait for the pages in flight
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
#pragma unroll
    for (int jj = 0; jj < 4; ++jj) {
      const uint4 w = (c < G) ? *(const uint4*)(s_q + c * kHd + 32 * jj + 8 * g) : make_uint4(0, 0, 0, 0);
      qb[jj] = __builtin_bit_cast(bf16x8_t, w);
    }
  }
  constexpr std::false_type kMid{};
  constexpr std::true_type kTail{};
  // The scheduling barriers keep the order below: left free, the scheduler
  // hoists the next page's score MFMAs above this page's, so every round
  // began by waiting for both pages in flight (vmcnt(0)) and issued its
  // next request only after that.
  for (; p + 16 < end; p += 12) {  // steady state: every request is a real page
    load_page(p + 8, r2);
    __builtin_amdgcn_sched_barrier(0);
    page_compute(p, r0, kMid);
    __builtin_amdgcn_sched_barrier(0);
    load_page(p + 12, r0);
    __builtin_amdgcn_sched_barrier(0);
    page_compute(p + 4, r1, kMid);
    __builtin_amdgcn_sched_barrier(0);
    load_page(p + 16, r1);
    __builtin_amdgcn_sched_barrier(0);
    page_compute(p + 8, r2, kMid);
    __builtin_amdgcn_sched_barrier(0);
  }
  if (p < end) {  // at most four pages left: p, p + 4, p + 8, p + 12
    if (p + 8 < end) load_page(p + 8, r2);
    page_compute(p, r0, kTail);
    if (p + 4 < end) {
      if (p + 12 < end) load_page(p + 12, r0);
      page_compute(p + 4, r1, kTail);
      if (p + 8 < end) {
        page_compute(p + 8, r2, kTail);
        if (p + 12 < end) page_compute(p + 12, r0, kTail);
      }
    }
  }
  // per-head normaliser: sum the four lane groups
  l += __shfl_xor(l, 16);
  l += __shfl_xor(l, 32);

  // merge the four waves through LDS
  __shared__ float s_acc[4][G][kHd];
  __shared__ float s_m[4][16], s_l[4][16];
  if (lane < 16) {
    s_m[wave][lane] = m;
    s_l[wave][lane] = l;
  }
#pragma unroll
  for (int blk = 0; blk < 8; ++blk)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int head = 4 * g + r;
      if (head < G) s_acc[wave][head][16 * blk + c] = acc[blk][r];
    }
  __syncthreads();
  // a sequence in one split is finished here (the combine's sums over one part
  // are exact: weight 2^0)
  const bool whole = it.part < 0;
  const long part = (long)it.part * n_kv + kvh;
  for (int e = threadIdx.x; e < G * kHd; e += 256) {
    const int head = e / kHd, dim = e - head * kHd;
    float M = fmaxf(fmaxf(s_m[0][head], s_m[1][head]), fmaxf(s_m[2][head], s_m[3][head]));
    float o = 0.f, L = 0.f;
#pragma unroll
    for (int w = 0; w < 4; ++w) {
      const float f = (s_m[w][head] == -INFINITY) ? 0.f : exp2f(s_m[w][head] - M);
      o += s_acc[w][head][dim] * f;
      L += s_l[w][head] * f;
    }
    if (whole) {
      out[((long)it.b * n_q + kvh * G + head) * kHd + dim] = f2bf(o / L);
      continue;
    }
    part_o[(part * G + head) * kHd + dim] = o;
    if (dim == 0) {
      part_ml[(part * G + head) * 2 + 0] = M;
      part_ml[(part * G + head) * 2 + 1] = L;
    }
  }
  __syncthreads();  // the next item reuses s_acc, s_m, s_l
  }
}

// o[b, head, :] = sum_s o_s 2^(m_s - M) / sum_s l_s 2^(m_s - M), splits in order.
__global__ __launch_bounds__(128) void decode_combine_kernel(const float* __restrict__ part_o,
                                                             const float* __restrict__ part_ml,
                                                             const int32_t* __restrict__ part_begin,
                                                             const int32_t* __restrict__ part_count,
                                                             bf16_t* __restrict__ o, int n_kv, int G) {
  const int b = blockIdx.x, head = blockIdx.y, dim = threadIdx.x;
  const int kvh = head / G, hg = head - kvh * G;
  const int p0 = part_begin[b], np = part_count[b];
  if (np == 1) return;  // written by the attention kernel
  const long stride = (long)n_kv * G;  // between consecutive splits of one (sequence, head)
  const long pi0 = ((long)p0 * n_kv + kvh) * G + hg;
  // Loads go four splits at a time so that their latencies overlap; the
  // arithmetic is the same sequence in split order as one split at a time.
  float M = -INFINITY;
  int i = 0;
  for (; i + 4 <= np; i += 4) {
    float mm[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) mm[u] = part_ml[(pi0 + (i + u) * stride) * 2];
#pragma unroll
    for (int u = 0; u < 4; ++u) M = fmaxf(M, mm[u]);
  }
  for (; i < np; ++i) M = fmaxf(M, part_ml[(pi0 + i * stride) * 2]);
  float acc = 0.f, L = 0.f;
  i = 0;
  for (; i + 4 <= np; i += 4) {
    float ov[4], mv[4], lv[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const long pi = pi0 + (i + u) * stride;
      ov[u] = part_o[pi * kHd + dim];
      mv[u] = part_ml[pi * 2];
      lv[u] = part_ml[pi * 2 + 1];
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const float f = exp2f(mv[u] - M);
      acc += ov[u] * f;
      L += lv[u] * f;
    }
  }
  for (; i < np; ++i) {
    const long pi = pi0 + i * stride;
    const float f = exp2f(part_ml[pi * 2] - M);
    acc += part_o[pi * kHd + dim] * f;
    L += part_ml[pi * 2 + 1] * f;
  }
  o[((long)b * n_kv * G + head) * kHd + dim] = f2bf(acc / L);
}

int launch_decode_attn(int G, int n_items, int n_kv, int n_seqs, const void* q, void* pool_layer,
                       const SeqInfo* si, const int32_t* bt, const DecodeItem* items, float* part_o,
                       float* part_ml, const int32_t* part_begin, const int32_t* part_count, void* o,
                       float scale_log2, hipStream_t st, int max_wg, const DecodeRope* rope) {
  if (n_seqs == 0) return 0;
  if (n_items > kMaxDecodeItems) return -1;
  int gy = n_items;
  if (max_wg > 0) gy = std::max(1, std::min(n_items, max_wg / n_kv));
  dim3 grid(n_kv, gy);
  const DecodeRope rp = rope ? *rope : DecodeRope{};
  if (rp.splits > 1 && rp.splits != 2 && rp.splits != 3 && rp.splits != 4 && rp.splits != 8) return -1;
#define PS_DECODE_GO(G_, ROPE_)                                                                                  \
  hipLaunchKernelGGL((decode_attn_kernel<G_, ROPE_>), grid, dim3(256), 0, st, (const bf16_t*)q,                 \
                     (bf16_t*)pool_layer, si, bt, items, part_o, part_ml, (bf16_t*)o, n_kv, n_items,          \
                     scale_log2, rp);
#define PS_DECODE_G(G_)                    \
  if (rp.splits) PS_DECODE_GO(G_, true)    \
  else PS_DECODE_GO(G_, false)
  switch (G) {
    case 1: PS_DECODE_G(1) break;
    case 2: PS_DECODE_G(2) break;
    case 4: PS_DECODE_G(4) break;
    case 8: PS_DECODE_G(8) break;
    case 16: PS_DECODE_G(16) break;
    default: return -1;
  }
#undef PS_DECODE_G
#undef PS_DECODE_GO
  if (n_items == n_seqs) return 0;  // every sequence in one split
  hipLaunchKernelGGL(decode_combine_kernel, dim3(n_seqs, n_kv * G), dim3(kHd), 0, st, part_o, part_ml,
                     part_begin, part_count, (bf16_t*)o, n_kv, G);
  return 0;
}

// ---------------------------------------------------------------- generic
// Vector-ALU attention for fp32 layers and for head sizes or groups the MFMA
// kernels do not take (any even head_dim <= 128): one workgroup per (row,
// query head), fp32 online softmax. A wave takes 64 keys (four pages) at a
// time: lane = key for the scores (each lane reads its key's row, q comes from
// LDS), one wave-wide max and sum per 64 keys, then lane = dimension for P V
// (each lane reads its dimension's 16 tokens of a V^T page, P comes from LDS).
// What bounds it is the chain of dependent loads and reductions, so the WK
// waves of a workgroup walk key blocks w, w + WK, ... side by side and merge
// in wave order. Tiny fp32 layer (4 sequences x 4 heads): one key at a time
// took 62 us at 144 keys, this 6.8; 512 causal rows 85 us, now 14.
template <typename T>
__device__ __forceinline__ float4 ld4(const T* p);
template <>
__device__ __forceinline__ float4 ld4<float>(const float* p) { return *(const float4*)p; }
template <>
__device__ __forceinline__ float4 ld4<bf16_t>(const bf16_t* p) {
  const uint2 w = *(const uint2*)p;
  return make_float4(bf_lo(w.x), bf_hi(w.x), bf_lo(w.y), bf_hi(w.y));
}

// ROPE (one new token per row, row r sequence r's): q is the QKV projection. The
// workgroup rotates its query head and the new key itself; the new token enters
// the softmax from LDS, and the first head of each group writes it to the pool,
// where no workgroup of the launch reads that slot. Saves a launch of 3.5 us on
// the stream and 2.3 on the host. Arithmetic of the rotation as in
// rope_kvwrite_kernel.
template <typename T, int WK, bool VEC, bool ROPE>  // VEC: head_dim a multiple of 4
__global__ __launch_bounds__(64 * WK) void attn_generic_kernel(const T* __restrict__ q, T* __restrict__ pool,
                                                               const SeqInfo* __restrict__ si,
                                                               const int32_t* __restrict__ bt, T* __restrict__ o,
                                                               int row0, int n_seqs, int n_q, int n_kv, int hd,
                                                               float scale, const double* __restrict__ inv_freq) {
  const int row = row0 + blockIdx.x, head = blockIdx.y;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  int lo = ROPE ? row : 0, hi = ROPE ? row : n_seqs - 1;
  while (lo < hi) {
    int mid = (lo + hi + 1) >> 1;
    if (si[mid].row_start <= row) lo = mid; else hi = mid - 1;
  }
  const SeqInfo s = si[lo];
  const int pos = s.kv_before + (row - s.row_start);
  const int kvh = head / (n_q / n_kv);
  const int32_t* btr = bt + s.bt_off;
  const long page_elts = 2L * kPageTokens * hd;
  __shared__ __attribute__((aligned(16))) float s_q[128], s_p[WK][64];
  __shared__ float s_o[WK][128], s_m[WK], s_l[WK];
  const int last = ROPE ? pos - 1 : pos;  // last key read from the pool
  float m = -INFINITY, l = 0.f, acc[2] = {0.f, 0.f};
  if constexpr (ROPE) {
    __shared__ float s_k[128], s_v[128];
    const int half = hd >> 1;
    const T* xr = q + (long)row * (n_q + 2 * n_kv) * hd;
    for (int u = threadIdx.x; u < 2 * hd; u += 64 * WK) {
      if (u < hd) {  // pair j of the query head, then of the new key
        const int j = u < half ? u : u - half;
        const T* x = xr + (u < half ? head : n_q + kvh) * hd + j;
        const float x1 = Elt<T>::load(x, 0), x2 = Elt<T>::load(x, half);
        double sd, cd;
        sincos((double)pos * inv_freq[j], &sd, &cd);
        float y1, y2;
        rope_pair(x1, x2, (float)cd, (float)sd, y1, y2);
        float* y = u < half ? s_q : s_k;
        y[j] = y1;
        y[j + half] = y2;
      } else {
        s_v[u - hd] = Elt<T>::load(xr, (n_q + n_kv + kvh) * hd + u - hd);
      }
    }
    __syncthreads();
    if (head % (n_q / n_kv) == 0) {
      T* pg = pool + ((long)btr[pos / kPageTokens] * n_kv + kvh) * page_elts;
      const int slot = pos % kPageTokens;
      for (int d = threadIdx.x; d < hd; d += 64 * WK) {
        Elt<T>::store(pg, (long)slot * hd + d, s_k[d]);
        Elt<T>::store(pg, (long)kPageTokens * hd + (long)d * kPageTokens + slot, s_v[d]);
      }
    }
    if (wave == 0) {  // wave 0 starts from the new token
      float sc = lane < hd ? s_q[lane] * s_k[lane] : 0.f;
      if (lane + 64 < hd) sc = fmaf(s_q[lane + 64], s_k[lane + 64], sc);
      for (int off = 32; off > 0; off >>= 1) sc += __shfl_xor(sc, off);
      m = sc * scale;
      l = 1.f;
      acc[0] = lane < hd ? s_v[lane] : 0.f;
      acc[1] = lane + 64 < hd ? s_v[lane + 64] : 0.f;
    }
  } else {
    for (int d = threadIdx.x; d < hd; d += 64 * WK) s_q[d] = Elt<T>::load(q, ((long)row * n_q + head) * hd + d);
    __syncthreads();
  }
  for (int k0 = wave * 64; k0 <= last; k0 += 64 * WK) {
    const int key = min(k0 + lane, last);
    const T* kr = pool + ((long)btr[key / kPageTokens] * n_kv + kvh) * page_elts + (long)(key % kPageTokens) * hd;
    float sc;
    if constexpr (VEC) {
      float4 d4 = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll 8
      for (int d = 0; d < hd; d += 4) {
        const float4 kv = ld4<T>(kr + d), qv = *(const float4*)(s_q + d);
        d4.x = fmaf(qv.x, kv.x, d4.x);
        d4.y = fmaf(qv.y, kv.y, d4.y);
        d4.z = fmaf(qv.z, kv.z, d4.z);
        d4.w = fmaf(qv.w, kv.w, d4.w);
      }
      sc = (d4.x + d4.y) + (d4.z + d4.w);
    } else {
      sc = 0.f;
      for (int d = 0; d < hd; ++d) sc = fmaf(s_q[d], Elt<T>::load(kr, d), sc);
    }
    sc = k0 + lane <= last ? sc * scale : -INFINITY;
    float mx = sc;
    for (int off = 32; off > 0; off >>= 1) mx = fmaxf(mx, __shfl_xor(mx, off));
    const float m_new = fmaxf(m, mx);
    const float base = m_new == -INFINITY ? 0.f : m_new;  // only scores of -inf yet: their weights are 0, not NaN
    const float alpha = expf(m - base), p = expf(sc - base);
    float ps = p;
    for (int off = 32; off > 0; off >>= 1) ps += __shfl_xor(ps, off);
    l = l * alpha + ps;
    m = m_new;
    // this wave's P values to its own LDS row, read back by the wave's other lanes
    s_p[wave][lane] = p;
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    acc[0] *= alpha;
    acc[1] *= alpha;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int kp = k0 + j * kPageTokens;
      if (kp > last) break;
      const int valid = last - kp + 1;  // tokens of the page that hold written keys, where < 16
      const T* vb = pool + ((long)btr[kp / kPageTokens] * n_kv + kvh) * page_elts + (long)kPageTokens * hd;
#pragma unroll
      for (int e = 0; e < 2; ++e) {
        const int dim = lane + 64 * e;
        if (dim >= hd) continue;
        float a = 0.f;
#pragma unroll
        for (int c = 0; c < 4; ++c) {
          const float4 v = ld4<T>(vb + (long)dim * kPageTokens + 4 * c), pv = *(const float4*)(&s_p[wave][16 * j + 4 * c]);
          a = fmaf(pv.x, 4 * c + 0 < valid ? v.x : 0.f, a);
          a = fmaf(pv.y, 4 * c + 1 < valid ? v.y : 0.f, a);
          a = fmaf(pv.z, 4 * c + 2 < valid ? v.z : 0.f, a);
          a = fmaf(pv.w, 4 * c + 3 < valid ? v.w : 0.f, a);
        }
        acc[e] += a;
      }
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  }
  if (lane == 0) {
    s_m[wave] = m;
    s_l[wave] = l;
  }
#pragma unroll
  for (int e = 0; e < 2; ++e) s_o[wave][lane + 64 * e] = acc[e];
  __syncthreads();
  for (int dim = threadIdx.x; dim < hd; dim += 64 * WK) {
    float M = s_m[0];  // wave 0 always has keys
    for (int w = 1; w < WK; ++w) M = fmaxf(M, s_m[w]);
    float L = 0.f, v = 0.f;
    for (int w = 0; w < WK; ++w) {
      if (w > 0 && w * 64 > last) break;  // waves past the last key took none
      const float f = expf(s_m[w] - M);
      L += s_l[w] * f;
      v += s_o[w][dim] * f;
    }
    Elt<T>::store(o, ((long)row * n_q + head) * hd + dim, v / L);
  }
}

int launch_attn_generic(int dt, int row0, int rows, int n_seqs, int n_q, int n_kv, int hd, const void* q,
                        const void* pool_layer, const SeqInfo* si, const int32_t* bt, void* o, float scale,
                        hipStream_t st) {
  if (rows == 0) return 0;
  if (hd > 128) return -1;
  dim3 grid(rows, n_q);
  auto go = [&](auto tag, auto wk, auto vec) {
    using T = decltype(tag);
    constexpr int WK = decltype(wk)::value;
    hipLaunchKernelGGL((attn_generic_kernel<T, WK, decltype(vec)::value, false>), grid, dim3(64 * WK), 0, st,
                       (const T*)q, (T*)pool_layer, si, bt, (T*)o, row0, n_seqs, n_q, n_kv, hd, scale, nullptr);
  };
  auto by_shape = [&](auto tag) {
    using W4 = std::integral_constant<int, 4>;
    using W16 = std::integral_constant<int, 16>;
    // few (row, head) pairs: 16 waves each, 1024 keys side by side
    const bool few = (long)rows * n_q <= 256;
    if (hd % 4 == 0) {
      if (few) go(tag, W16{}, std::true_type{});
      else go(tag, W4{}, std::true_type{});
    } else {
      if (few) go(tag, W16{}, std::false_type{});
      else go(tag, W4{}, std::false_type{});
    }
  };
  if (dt == 1) by_shape(bf16_t{});
  else by_shape(float{});
  return 0;
}

int launch_attn_generic_rope(int rows, int n_q, int n_kv, int hd, const float* qkv, void* pool_layer, const SeqInfo* si,
                             const int32_t* bt, const double* inv_freq, float* o, float scale, hipStream_t st) {
  if (rows == 0) return 0;
  if (hd > 128 || hd % 2) return -1;
  auto go = [&](auto wk, auto vec) {
    constexpr int WK = decltype(wk)::value;
    hipLaunchKernelGGL((attn_generic_kernel<float, WK, decltype(vec)::value, true>), dim3(rows, n_q), dim3(64 * WK), 0, st,
                       qkv, (float*)pool_layer, si, bt, o, 0, rows, n_q, n_kv, hd, scale, inv_freq);
  };
  using W4 = std::integral_constant<int, 4>;
  using W16 = std::integral_constant<int, 16>;
  const bool few = (long)rows * n_q <= 256;  // as launch_attn_generic
  if (hd % 4 == 0) {
    if (few) go(W16{}, std::true_type{});
    else go(W4{}, std::true_type{});
  } else {
    if (few) go(W16{}, std::false_type{});
    else go(W4{}, std::false_type{});
  }
  return 0;
}

}  // namespace ps
