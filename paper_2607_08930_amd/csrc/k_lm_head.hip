// Output head fused with confidence-aware parallel decoding (paragraph
// "Vectorized mixed-schedule execution"; the greedy parallel decoding of
// Fast-dLLM, "Implementation details"). The logit of vocabulary entry v at a
// masked block position is the inner product of the position's final hidden
// state with row v of the output-head matrix. The logits are reduced to
// (max, smallest index attaining it, sum of exp(x - max)) as they leave the
// matrix cores and are never stored; the selection then runs unchanged.
//
// k_lm_pack   once per model: lays the output-head matrix out as the
//             contiguous 16 KiB slabs the ring stages copy (the [V][d] layout
//             would read 64 bytes from each of 256 rows 2 d bytes apart).
// k_lm_rows   one workgroup lists the masked rows (j < B_i, masked) of the
//             compact [n][L] block state in increasing order and counts them.
// k_lm_head   C^T = W H^T on v_mfma_f32_32x32x16_bf16 over 256 (vocabulary)
//             x 64, 128, 192 or 256 (listed rows) tiles; K moves HBM -> LDS
//             in 32-wide slices through a ring by direct DMA. Vocabulary is the MFMA M
//             axis, so a lane holds one row's column of 16 logits per 32x32
//             block: the epilogue reduces 32 logits per lane and row, exchanges
//             once with the other half-wave and once through LDS. One DecPartial per (row,
//             128-entry vocabulary slice).
// k_lm_merge  one workgroup per listed row merges its slices into the DecPartial
//             the selection reads.
#include <float.h>
#include <limits.h>

#include "bs_internal.h"
#include "bs_lds.h"

namespace bs {
namespace {

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef float f32x16_t __attribute__((ext_vector_type(16)));
constexpr float kLog2e = 1.4426950408889634f;

// Latency-bound (one workgroup): the flags of 4096 positions are loaded
// at once and counted by ballots, so that a batch of up to 4096 positions waits
// for one round trip to memory and one barrier: shortest launches of 256
// positions 4.3 -> 3.1 us, of 2048 positions 4.9 -> 3.8 us (a serial count and a
// scan of 1024 threads by doubling, before).
__global__ __launch_bounds__(1024) void k_lm_rows(LmArgs a) {
  constexpr int NC = 4;                     // chunks of 1024 positions per trip
  __shared__ int cnt[2][NC * 16];           // listed positions of (chunk, wave), by trip parity
  const int total = a.n * a.L, t = threadIdx.x, w = t >> 6, lane = t & 63;
  int pos = 0, trip = 0;
  for (int x0 = 0; x0 < total; x0 += NC * 1024, trip ^= 1) {
    bool on[NC];
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      const int x = min(x0 + c * 1024 + t, total - 1);
      const int i = x / a.L, j = x - i * a.L;
      const bs_req_desc r = a.reqs[i];
      const uint8_t m = a.masked[x];
      on[c] = x0 + c * 1024 + t < total && j < geo_of(r, a.L).B && m != 0;
    }
    unsigned long long bits[NC];
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      bits[c] = __ballot(on[c]);
      if (lane == 0) cnt[trip][c * 16 + w] = __popcll(bits[c]);
    }
    __syncthreads();
    int sum = cnt[trip][lane];              // NC * 16 == 64: inclusive scan over (chunk, wave)
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const int v = __shfl_up(sum, o, 64);
      if (lane >= o) sum += v;
    }
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      const int before = __shfl(sum, max(c * 16 + w - 1, 0), 64);
      if (on[c]) a.rows[pos + (c * 16 + w ? before : 0) + __popcll(bits[c] & ((1ull << lane) - 1))] = x0 + c * 1024 + t;
    }
    pos += __shfl(sum, 63, 64);
  }
  if (t == 0) *a.count = pos;
}

// LDS rows hold 32 bf16 of K (64 bytes, four 16-byte chunks). Chunk c of tile
// row r sits in slot c ^ ((r >> 2) & 3): the 32 rows one MFMA operand read
// touches then spread two per bank group.
constexpr int kTile = kLmNT * kLmKT;        // elements of the W tile of a stage: 16 KiB
constexpr int kLdsBytes = 160 * 1024;       // all of a CU's LDS: one workgroup per CU

template <int I>
struct Const {
  static constexpr int value = I;
};

// Wait until at most k (uniform, 0 <= k <= K) stages of C transfers each are
// outstanding. In the loop k = K but for its last stages.
template <int C, int K>
__device__ inline void wait_stages(int k) {
  if (k >= K) {
    wait_vm_c<K * C>();
  } else if constexpr (K > 0) {
    wait_stages<C, K - 1>(k);
  }
}

// One workgroup tile: 256 vocabulary entries x 64 M listed rows, M = 1..4, in
// stages of KS slices of the contraction (each 32 wide).
// Wave (wv, wr) = (w >> 1, w & 1) computes vocabulary rows 64 wv .. + 64 (two
// 32-row blocks) x listed rows 32 M wr .. + 32 M.
//
// The matrix cores bound it, at the clock that their power leaves: the
// operands of each half of a K slice (16 of its 32) are read from LDS beside
// the MFMAs of the half before, and the stage's one barrier stands before its
// last half, so that a wave leaves it with its next operands in registers and
// the slot that the barrier frees is refilled at once. The order is fixed by
// scheduling fences: one MFMA, then one LDS read or one transfer.
// Measured on a Dream-7B head (V = 152064, d = 3584), 1035 listed rows: 1065 us,
// MFMA busy 60% at 1.75 GHz. With a barrier before the reads of a whole slice
// and five 256-row tiles the same rows took 1640 us. Four waves of 128 x 32 M
// (two thirds of the LDS reads, accumulators in AGPRs, one wave per SIMD) took
// 12% longer than eight.
//
// KS = 2 where a slice has few MFMAs between barriers (M <= 2 and d a multiple of
// 64): 125 rows of a LLaDA-8B head 206 -> 196 us (this kernel). At M = 3 and 4 it leaves two
// stages of LDS and takes longer: 502 rows 492 -> 526, 1035 of a Dream-7B head
// 1088 -> 1125.
//
// ONCE: W is read by one row tile only and streams past the L2's other lines
// with the non-temporal hint (calls on a LLaDA-8B head: 12 rows 193 -> 174 us, 64:
// 193 -> 177, 125: 216.7 -> 212; Dream-7B head, 52 rows: 224 -> 208). Matrices of
// less than the 256 MB Infinity Cache, too: between two calls a serving program
// streams its layers, so W comes from memory (4 requests, 32 MB: 55.5 -> 51.4, 65
// MB: 48.0 -> 42.1, 262 MB: 105.8 -> 84.1). Called back to back with nothing between,
// W stays in that cache and the plain form is the faster by up to a quarter
// (65 MB: 34.7 against 32.7, 262 MB: 76.1 against 58.6).
template <int M, bool ONCE, int KS>
__device__ inline void lm_tile(const LmArgs& a, uint16_t* ring, int vt, int r0, int count) {
  constexpr int HB = 4 * M;                              // 1 KiB blocks (16 rows) of the H tile
  constexpr int HT = HB * 512;                           // elements of the H tile of a slice
  constexpr int SLOT = KS * (kTile + HT);                // elements of a stage: KS W tiles, then KS H tiles
  constexpr int NS = kLdsBytes / (SLOT * 2);             // 5 stages at M = 4, 3 (of two slices) at M = 2
  constexpr int CHI = KS * (2 + (HB + 7) / 8), CLO = KS * (2 + HB / 8);   // transfers per stage of waves 0..3 and 4..7
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;

  // DMA: wave w issues W blocks 2w and 2w + 1 and H blocks w and w + 8 (where
  // the tile has them). W comes from the packed slabs (already in LDS order:
  // a block is one contiguous KiB). H rows are gathered through the row list:
  // lane l fills slot l & 3 of tile row 16 b + (l >> 2) with global chunk
  // (l & 3) ^ ((l >> 4) & 3).
  const uint16_t* hp[2];
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    const int row = 16 * (w + 8 * q) + (lane >> 2);
    hp[q] = a.hidden + (int64_t)a.rows[min(r0 + row, count - 1)] * a.d + ((lane & 3) ^ ((lane >> 4) & 3)) * 8;
  }
  const uint32_t lds0 = lds_addr(ring);
  const uint16_t* wp = a.w + (int64_t)vt * (a.d / kLmKT) * kTile + w * 1024;   // next stage to issue
  uint32_t fill = lds0;                                                        // and its slot
  auto issue_w = [&](int k, int q) {                     // slice k of the stage
    const uint64_t src = uniform64(wp + k * kTile + q * 512);
    if constexpr (ONCE)
      dma16_sv_once(fill + k * kTile * 2 + (2 * w + q) * 1024, src, (uint32_t)(lane * 16));
    else
      dma16_sv(fill + k * kTile * 2 + (2 * w + q) * 1024, src, (uint32_t)(lane * 16));
  };
  auto issue_h = [&](int k, int q) {
    if (HB >= 8 * (q + 1) || (HB > 8 * q && w < 4))
      dma16(fill + (KS * kTile + k * HT) * 2 + (w + 8 * q) * 1024, hp[q] + k * kLmKT);
  };
  auto issued = [&] {
    wp += KS * kTile;
    hp[0] += KS * kLmKT;
    hp[1] += KS * kLmKT;
    fill = fill + SLOT * 2 == lds0 + NS * SLOT * 2 ? lds0 : fill + SLOT * 2;
  };
  auto wait_ahead = [&](int k) {
    if (CHI == CLO || w < 4)
      wait_stages<CHI, NS - 1>(k);
    else
      wait_stages<CLO, NS - 1>(k);
  };
  auto barrier = [] {
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
  };

  // MFMA operands: lane (g, n) reads row n of a 32-row block, chunk 2 s + g of
  // the slice's half s.
  const int g = lane >> 5, n = lane & 31;
  const int wv = w >> 1, wr = w & 1;
  int off[2];
#pragma unroll
  for (int s = 0; s < 2; ++s) off[s] = n * kLmKT + (((2 * s + g) ^ ((n >> 2) & 3)) * 8);
  f32x16_t acc[2][M];
#pragma unroll
  for (int vb = 0; vb < 2; ++vb)
#pragma unroll
    for (int rb = 0; rb < M; ++rb)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[vb][rb][r] = 0.0f;
  bf16x8_t F[2][2 + M];                                  // per half: two W fragments, M H fragments
  auto read = [&](const uint16_t* st, int hs, int i) {   // half hs of the stage's 2 KS
    const int k = hs >> 1, s = hs & 1;
    const uint16_t* p = i < 2 ? st + k * kTile + (64 * wv + 32 * i) * kLmKT
                              : st + KS * kTile + k * HT + (32 * M * wr + 32 * (i - 2)) * kLmKT;
    F[s][i] = *reinterpret_cast<const bf16x8_t*>(p + off[s]);
  };

  const int nk = a.d / (kLmKT * KS);                     // stages
  for (int t = 0; t < min(NS, nk); ++t) {
#pragma unroll
    for (int k = 0; k < KS; ++k) {
      issue_w(k, 0);
      issue_w(k, 1);
      issue_h(k, 0);
      issue_h(k, 1);
    }
    issued();
  }
  wait_ahead(min(NS, nk) - 1);
  barrier();
  const uint16_t* st = ring;
#pragma unroll
  for (int i = 0; i < 2 + M; ++i) read(st, 0, i);

  // Half hs of stage t: 2 M MFMAs on F[hs & 1]; beside them the reads of the next
  // half (of the stage at `next`), and in the last half the transfers of stage t + NS.
  auto half = [&](auto half_tag, auto refill_tag, const uint16_t* next) {
    constexpr int hs = decltype(half_tag)::value, refill = decltype(refill_tag)::value;
    constexpr int s = hs & 1, nx = (hs + 1) % (2 * KS);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 0; i < 2 * M; ++i) {
      acc[i & 1][i >> 1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(F[s][i & 1], F[s][2 + (i >> 1)], acc[i & 1][i >> 1], 0, 0, 0);
      if (i < 2 + M) read(next, nx, i);
      if (i == 2 * M - 1) {
#pragma unroll
        for (int k = 2 * M; k < 2 + M; ++k) read(next, nx, k);      // M = 1: three reads, two MFMAs
      }
      if (refill && nx == 0 && i >= 2 * M - 2) {
#pragma unroll
        for (int k = 0; k < KS; ++k) {
          issue_w(k, i & 1);
          issue_h(k, i & 1);
        }
      }
      __builtin_amdgcn_sched_barrier(0);
    }
    if (refill && nx == 0) issued();
  };
  auto stage = [&](int t, auto refill_tag) {
    half(Const<0>{}, refill_tag, st);
    if constexpr (KS == 2) {
      half(Const<1>{}, refill_tag, st);
      half(Const<2>{}, refill_tag, st);
    }
    // Stage t + 1 has landed once only later ones are in flight. Past the
    // barrier every wave holds its last operands of stage t, so its slot is free.
    wait_ahead(refill_tag.value ? NS - 2 : max(nk - 2 - t, 0));
    barrier();
    st = st + SLOT == ring + NS * SLOT ? ring : st + SLOT;
    // after the last stage this reads a slot that nobody refills; the operands are not used
    half(Const<2 * KS - 1>{}, refill_tag, st);
  };
  int t = 0;
  for (; t + NS < nk; ++t) stage(t, Const<1>{});
  for (; t < nk; ++t) stage(t, Const<0>{});

  // Epilogue: lane (g, n) holds C^T[vocab v][row n] for
  // v = v0 + 64 wv + 32 vb + 8 (r / 4) + 4 g + r % 4.
  const int v0 = vt * kLmNT;
  const int vbase = v0 + 64 * wv + 4 * g;
  if (v0 + kLmNT > a.V) {                      // ragged last vocabulary tile only
#pragma unroll
    for (int vb = 0; vb < 2; ++vb)
#pragma unroll
      for (int r = 0; r < 16; ++r)
        if (vbase + 32 * vb + 8 * (r >> 2) + (r & 3) >= a.V) {
#pragma unroll
          for (int rb = 0; rb < M; ++rb) acc[vb][rb][r] = -__builtin_inff();
        }
  }
  barrier();                                   // the ring is read no more
  DecPartial* part = reinterpret_cast<DecPartial*>(ring);   // [4][64 M]: one per (wv, listed row of the tile)
#pragma unroll
  for (int rb = 0; rb < M; ++rb) {
    float mx = -__builtin_inff();
    int am = INT_MAX;
#pragma unroll
    for (int vb = 0; vb < 2; ++vb)
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const float x = acc[vb][rb][r];
        const int id = vbase + 32 * vb + 8 * (r >> 2) + (r & 3);
        if (x > mx || (x == mx && id < am)) {
          mx = x;
          am = id;
        }
      }
    const float mo = __shfl_xor(mx, 32, 64);
    const int ao = __shfl_xor(am, 32, 64);
    const float mm = fmaxf(mx, mo);
    int A = mx == mm ? am : INT_MAX;
    if (mo == mm) A = min(A, ao);
    const float nm = mm == -__builtin_inff() ? 0.0f : -mm * kLog2e;   // a slice past V sums to 0
    float sum = 0.0f;
#pragma unroll
    for (int vb = 0; vb < 2; ++vb)
#pragma unroll
      for (int r = 0; r < 16; ++r) sum += __builtin_amdgcn_exp2f(fmaf(acc[vb][rb][r], kLog2e, nm));
    sum += __shfl_xor(sum, 32, 64);
    if (g == 0) {
      DecPartial p;
      p.m = mm;
      p.s = sum;
      p.a = A;
      p.pad = 0;
      part[wv * 64 * M + 32 * M * wr + 32 * rb + n] = p;
    }
  }
  barrier();
  // one thread per (listed row, 128-entry slice) joins the slice's two halves
  const int x = threadIdx.x >> 1, h = threadIdx.x & 1;
  if (x < 64 * M && r0 + x < count) {
    const DecPartial p0 = part[2 * h * 64 * M + x], p1 = part[(2 * h + 1) * 64 * M + x];
    DecPartial p;
    p.m = fmaxf(p0.m, p1.m);
    p.s = p.m == -__builtin_inff() ? p0.s + p1.s
                                   : p0.s * __builtin_amdgcn_exp2f((p0.m - p.m) * kLog2e) +
                                         p1.s * __builtin_amdgcn_exp2f((p1.m - p.m) * kLog2e);
    p.a = min(p0.m == p.m ? p0.a : INT_MAX, p1.m == p.m ? p1.a : INT_MAX);
    p.pad = 0;
    a.slices[(int64_t)(r0 + x) * a.parts + 2 * vt + h] = p;
  }
}

__global__ __launch_bounds__(512, 1) void k_lm_head(LmArgs a) {
  static_assert(kLmNT == 256 && kLmMT == 256 && kLmKT == 32, "tiling below assumes these");
  __shared__ __align__(1024) uint16_t ring[kLdsBytes / 2];
  const int count = *a.count;
  if (count == 0) return;
  const int nvt = (a.V + kLmNT - 1) / kLmNT;
  // The listed rows fall into units of 64, dealt evenly to the fewest row
  // tiles of at most four units: 1035 rows are tiles of 4, 4, 3, 3 and 3 units
  // (1088 rows) rather than five of 256 (1280), 125 rows one of 128. Whole
  // calls before and after, by rows: LLaDA-8B head 12: 276 -> 197 us, 125: 277
  // -> 220, 268: 517 -> 368, 502: 554 -> 493; Dream-7B head 1035: 1673 -> 1071.
  const int units = (count + 63) / 64;
  const int nact = (units + 3) / 4, base = units / nact, extra = units - base * nact;
  // Workgroups b = x + 8 q run on XCD x. Consecutive q on one XCD take all row
  // tiles of one vocabulary tile, which then share that XCD's L2 copy of the W
  // slab (W is read about once; the hidden rows come from L2 or the Infinity
  // Cache), and the XCDs take the vocabulary tiles in turn. One row tile per
  // XCD took 403 us on 268 rows (two row tiles), a contiguous range of
  // vocabulary tiles per XCD 230 us on 125 rows.
  const int x = (int)(blockIdx.x & 7), q = (int)(blockIdx.x >> 3);
  const int vt = (q / nact) * 8 + x, rt = q % nact;
  if (vt >= nvt) return;
  const int r0 = 64 * (rt * base + min(rt, extra));
  auto tile = [&](auto once) {
    constexpr bool ONCE = decltype(once)::value != 0;
    auto go = [&](auto m) {
      constexpr int M = decltype(m)::value;
      if constexpr (M <= 2) {
        if (a.d % (2 * kLmKT) == 0) return lm_tile<M, ONCE, 2>(a, ring, vt, r0, count);
      }
      lm_tile<M, ONCE, 1>(a, ring, vt, r0, count);
    };
    switch (base + (rt < extra ? 1 : 0)) {
      case 1: go(Const<1>{}); break;
      case 2: go(Const<2>{}); break;
      case 3: go(Const<3>{}); break;
      default: go(Const<4>{}); break;
    }
  };
  if (nact == 1)
    tile(Const<1>{});
  else
    tile(Const<0>{});
}

__device__ inline float wave_max(float v) {
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) v = fmaxf(v, __shfl_xor(v, o, 64));
  return v;
}
__device__ inline float wave_sum(float v) {
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}
__device__ inline int wave_min_i(int v) {
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) v = min(v, __shfl_xor(v, o, 64));
  return v;
}

// One workgroup per listed row. Latency-bound: a thread's parts (five of the
// 1188 of a Dream-7B head) are loaded at once and kept, so that a row waits for
// one round trip to memory: 125 rows x 988 parts 12.4 -> 5.4 us, 1035 rows x
// 1188 parts 17.3 -> 7.2 us (one wave per row, two passes, before).
__global__ __launch_bounds__(256) void k_lm_merge(LmArgs a) {
  constexpr int NP = 8;
  const int x = blockIdx.x, t = threadIdx.x, w = t >> 6;
  if (x >= *a.count) return;
  const DecPartial* p = a.slices + (int64_t)x * a.parts;
  DecPartial q[NP];
#pragma unroll
  for (int k = 0; k < NP; ++k) {
    if (t + 256 * k < a.parts)
      q[k] = p[t + 256 * k];
    else
      q[k] = DecPartial{-__builtin_inff(), 0.0f, INT_MAX, 0};
  }
  float M = -__builtin_inff();
#pragma unroll
  for (int k = 0; k < NP; ++k) M = fmaxf(M, q[k].m);
  for (int k = t + 256 * NP; k < a.parts; k += 256) M = fmaxf(M, p[k].m);
  __shared__ float sm[4], ss[4];
  __shared__ int sa[4];
  M = wave_max(M);
  if ((t & 63) == 0) sm[w] = M;
  __syncthreads();
  M = fmaxf(fmaxf(sm[0], sm[1]), fmaxf(sm[2], sm[3]));
  float S = 0.0f;
  int A = INT_MAX;
  auto fold = [&](const DecPartial& v) {
    if (v.m != -__builtin_inff()) S += v.s * __builtin_amdgcn_exp2f((v.m - M) * kLog2e);
    if (v.m == M) A = min(A, v.a);
  };
#pragma unroll
  for (int k = 0; k < NP; ++k) fold(q[k]);
  for (int k = t + 256 * NP; k < a.parts; k += 256) fold(p[k]);
  S = wave_sum(S);
  A = wave_min_i(A);
  if ((t & 63) == 0) {
    ss[w] = S;
    sa[w] = A;
  }
  __syncthreads();
  if (t == 0) {
    DecPartial r;
    r.m = M;
    r.s = (ss[0] + ss[1]) + (ss[2] + ss[3]);
    r.a = min(min(sa[0], sa[1]), min(sa[2], sa[3]));
    r.pad = 0;
    a.row_part[a.rows[x]] = r;
  }
}

// One thread per 16-byte chunk of the packed matrix: slab (vt, kt), row r,
// slot s holds W[vt * 256 + r][32 kt + 8 (s ^ ((r >> 2) & 3)) .. + 8], or
// zeros for rows past V.
__global__ __launch_bounds__(256) void k_lm_pack(const uint16_t* w, int64_t ldw, int V, int d, uint16_t* packed) {
  const int64_t x = (int64_t)blockIdx.x * 256 + threadIdx.x;      // chunk index
  const int nkt = d / kLmKT;
  const int64_t total = (int64_t)((V + kLmNT - 1) / kLmNT) * nkt * kLmNT * 4;
  if (x >= total) return;
  const int slot = (int)(x & 3), r = (int)((x >> 2) & (kLmNT - 1));
  const int64_t slab = x >> 10;                                     // 1024 chunks per slab
  const int kt = (int)(slab % nkt), vt = (int)(slab / nkt);
  const int v = vt * kLmNT + r;
  v4u val = v4u{0u, 0u, 0u, 0u};
  if (v < V) val = ld16(w + (int64_t)v * ldw + kt * kLmKT + (slot ^ ((r >> 2) & 3)) * 8);
  st16(packed + x * 8, val);
}

}  // namespace

hipError_t launch_lm_pack(const uint16_t* w, int64_t ldw, int V, int d, uint16_t* packed, hipStream_t s) {
  const int64_t chunks = (int64_t)((V + kLmNT - 1) / kLmNT) * (d / kLmKT) * kLmNT * 4;
  hipLaunchKernelGGL(k_lm_pack, dim3((unsigned)((chunks + 255) / 256)), dim3(256), 0, s, w, ldw, V, d, packed);
  return hipGetLastError();
}

hipError_t launch_lm_rows(const LmArgs& a, hipStream_t s) {
  hipLaunchKernelGGL(k_lm_rows, dim3(1), dim3(1024), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_lm_gemm(const LmArgs& a, hipStream_t s) {
  const int nvt = (a.V + kLmNT - 1) / kLmNT;
  const int nrt = (a.n * a.L + kLmMT - 1) / kLmMT;
  const int per_xcd = (nvt + 7) / 8 * nrt;     // the row count is known on the device only
  hipLaunchKernelGGL(k_lm_head, dim3((unsigned)(8 * per_xcd)), dim3(512), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_lm_merge(const LmArgs& a, hipStream_t s) {
  hipLaunchKernelGGL(k_lm_merge, dim3((unsigned)(a.n * a.L)), dim3(256), 0, s, a);
  return hipGetLastError();
}

}  // namespace bs
