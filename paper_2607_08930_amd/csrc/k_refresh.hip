// Dual-cache refresh at a block start (the dual cache of Fast-dLLM that the
// paper integrates, Sections "Experimental setup" and "Diffusion LLM Inference
// Optimization"; position ids of paragraph "Logical positional alignment").
//
// The refresh forward recomputes the KV of every cell of a request's logical
// row and attends every position to the whole row (bidirectional). Per layer
// this file runs the two parts that do not need model weights:
//
// k_refresh_kv   rotary embedding of the keys at their position ids (the
//                count of real tokens before the cell, i.e. the cell's logical
//                position) and the scatter of rotated keys and plain values
//                from the token-major projections into the head-major cache.
//                HBM-bound: every byte is read once and written once.
// k_refresh_attn full-row attention over the refreshed cache, the queries
//                rotated as they are loaded. A workgroup of four waves owns
//                128 query positions of one head, 32 queries per wave
//                (32x32x16 MFMAs), and two workgroups share a CU (two waves
//                per SIMD), so one workgroup's prologue (first tiles, queries
//                and their rotation) runs beside the other's loop. K/V tiles
//                of 32 keys stream HBM/L2 -> LDS by direct DMA through a
//                4-stage ring. Inside a wave the loop is software-pipelined by
//                32-key sub-tiles: while the exponentials of sub-tile u run on
//                the VALU, the matrix core accumulates P V of u - 1 and
//                computes the scores of u + 1. Four sub-tiles are unrolled
//                over the ring's slots, so LDS addresses are immediates and a
//                sub-tile is 16 MFMAs beside 59 VALU instructions. What bounds
//                it: MFMA and VALU issue on long rows (64 Dream-7B-shaped rows:
//                matrix cores busy 46% at 1.8 GHz), each item's first tiles,
//                queries and output on short ones (32 LLaDA-8B-shaped rows: 30%
//                at 2.1 GHz). Measured on the former (1.17 TFLOP): 1.3 ms in
//                the mean of 56 launches and 1.2 in the fastest, 0.9 PFLOP/s;
//                with per-sub-tile address arithmetic (about 40 VALU
//                instructions more) and V fragments read right before their
//                MFMA, 1.11x the whole call's time.
#include "bs_lds.h"
#include "bs_refresh.h"

namespace bs {
namespace {

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4_t __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
typedef float f32x16_t __attribute__((ext_vector_type(16)));
typedef __attribute__((address_space(3))) bf16x4_t lds_bf16x4;

__device__ inline float bf16_lo(uint32_t w) { return __uint_as_float(w << 16); }
__device__ inline float bf16_hi(uint32_t w) { return __uint_as_float(w & 0xffff0000u); }
typedef float f32x2_t __attribute__((ext_vector_type(2)));
__device__ inline uint32_t pack_bf16(float lo, float hi) {
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2_t{lo, hi}, bf16x2_t));
}

// Rotate the feature pairs (x1[e], x2[e]) of 8 consecutive features f0 .. f0+7
// of the first half (partners f + D/2 in x2) by the angle pos * exp2(f * nl2b).
// The angle is formed in turns, pos * exp2(f * nl2b - log2(2 pi)); its
// fractional part (exact) feeds the hardware sine and cosine, which take
// turns. The fp32 roundings of the inverse frequency and of the product leave
// an angle error of a few 2^-23 relative, under 4e-4 rad for positions below
// 2048.
__device__ inline void rope8(v4u& x1, v4u& x2, int f0, float pos, float nl2b) {
  constexpr float kNegLog2TwoPi = -2.6514961294723187f;
#pragma unroll
  for (int w = 0; w < 4; ++w) {
    float a[2], b[2];
    a[0] = bf16_lo(x1[w]); a[1] = bf16_hi(x1[w]);
    b[0] = bf16_lo(x2[w]); b[1] = bf16_hi(x2[w]);
    float ya[2], yb[2];
#pragma unroll
    for (int e = 0; e < 2; ++e) {
      const float turns = pos * __builtin_amdgcn_exp2f(fmaf((float)(f0 + 2 * w + e), nl2b, kNegLog2TwoPi));
      const float fr = __builtin_amdgcn_fractf(turns);
      const float sn = __builtin_amdgcn_sinf(fr), cs = __builtin_amdgcn_cosf(fr);
      ya[e] = a[e] * cs - b[e] * sn;
      yb[e] = b[e] * cs + a[e] * sn;
    }
    x1[w] = pack_bf16(ya[0], ya[1]);
    x2[w] = pack_bf16(yb[0], yb[1]);
  }
}

// ------------------------------------------------------------------ keys/values
// Thread u of request blockIdx.y: cell t = u / (Hkv * HC), KV head c, and the
// 16-byte chunk pair (ch, ch + HC) of that head's row (features 8 ch .. + 7 and
// their rotation partners D/2 + 8 ch .. + 7).
template <int D>
__global__ __launch_bounds__(256) void k_refresh_kv(RefKvArgs a) {
  constexpr int HC = D / 16;
  const bs_req_desc r = a.reqs[blockIdx.y];
  const int len = r.p + r.g;
  const int u = blockIdx.x * 256 + threadIdx.x;
  if (u >= len * a.Hkv * HC) return;
  const int ch = u % HC, c = (u / HC) % a.Hkv, t = u / (HC * a.Hkv);
  const int64_t src = (((int64_t)r.row * a.W + r.off + t) * a.Hkv + c) * D + ch * 8;
  const int64_t dst = (((int64_t)r.row * a.Hkv + c) * a.W + r.off + t) * D + ch * 8;
  v4u k1 = ld16(a.k + src), k2 = ld16(a.k + src + D / 2);
  const v4u v1 = ld16(a.v + src), v2 = ld16(a.v + src + D / 2);
  if (a.rope) rope8(k1, k2, ch * 8, (float)t, a.nl2b);
  st16(a.k_cache + dst, k1);
  st16(a.k_cache + dst + D / 2, k2);
  st16(a.v_cache + dst, v1);
  st16(a.v_cache + dst + D / 2, v2);
}

// ------------------------------------------------------------------ attention
// XOR swizzle of a cache row's 16-byte slots in LDS (D = 128: 16 slots) for
// an LDS that serves 256 bytes (64 banks of 4 bytes) per cycle. The 32 lanes
// of one transposed V read cover rows r0 .. r0 + 3 (r0 % 4 == 0) at chunks
// 4 t .. 4 t + 3: row bits 0..1 move to slot bits 2..3, so those reads land
// in 16 distinct slots; row bits 2..3 move to slot bits 0..1, so any 16
// consecutive rows still get distinct slots for one chunk (the K reads).
__device__ inline int swz16(int row) { return ((row & 3) << 2) | ((row >> 2) & 3); }

__device__ inline float vmax(float x, float y) { return __builtin_elementwise_maximum(x, y); }

// lsum + the eight bf16 weights in p (the values the P V MFMA consumes)
__device__ inline float add_weights(float lsum, const bf16x8_t& p) {
  const bf16x2_t one = {(__bf16)1.0f, (__bf16)1.0f};
#pragma unroll
  for (int k = 0; k < 4; ++k) lsum = __builtin_amdgcn_fdot2_f32_bf16(bf16x2_t{p[2 * k], p[2 * k + 1]}, one, lsum, false);
  return lsum;
}

// compile-time integer passed to a generic lambda
template <int V>
struct Const {
  static constexpr int value = V;
  __device__ constexpr operator int() const { return V; }
};

// NW waves of 32 queries each share the K/V ring. Two 32-query blocks per wave
// would feed every LDS fragment to two MFMAs but need about 400 registers (one
// wave per SIMD, so nothing hides the softmax arithmetic and the LDS latency:
// 20% slower on the Dream-7B shape).
template <int D, int NW>
__global__ __launch_bounds__(64 * NW, 2) void k_refresh_attn(RefArgs a) {
  static_assert(D == 128, "the refresh attention is laid out for D = 128");
  static_assert(NW * 32 == kRefQ, "a workgroup covers kRefQ queries");
  constexpr int KT = kRefKT, NS = kRefNS;
  constexpr int NKK = D / 16;        // K-steps of a score MFMA
  constexpr int NDT = D / 32;        // 32-feature output tiles
  constexpr int TILE = KT * D;       // elements of one K (or V) tile
  constexpr int STAGE = 2 * TILE;    // K tile, then V tile
  constexpr int SPT = KT / 32;       // 32-key sub-tiles per tile
  constexpr int PB = STAGE * 2 / 1024 / NW;   // 1 KiB DMA blocks per stage and wave
  constexpr int WPT = NW / 2;        // waves per tensor (K, then V)
  __shared__ __align__(1024) uint16_t ring[NS * STAGE];

  const RefItem it = a.items[blockIdx.x];
  if (it.row < 0) return;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63, g = lane >> 5, n = lane & 31;
  const int len = it.len, h = it.h, c = h / a.G;
  const int ntiles = (len + KT - 1) / KT, nsub = (len + 31) / 32;
  const int qbase = it.q0 + 32 * w;             // first query of this wave
  const bool active = qbase < len;                   // wave-uniform

  const int64_t cache_off = (((int64_t)it.row * a.Hkv + c) * a.W + it.off) * D;
  const uint16_t* kcb = a.k_cache + cache_off;
  const uint16_t* vcb = a.v_cache + cache_off;

  // DMA: wave w moves PB blocks of a stage; the first NW/2 waves the K tile,
  // the others the V tile. Block rb of a tile covers its rows 4 rb .. + 3;
  // lane l fills row 4 rb + l / 16, slot l % 16, from global chunk
  // slot ^ swz(row).
  const int tensor = w / WPT;
  const uint16_t* tb_src = tensor ? vcb : kcb;
  // the ring holds NS K tiles, then NS V tiles, so that every LDS read is a
  // lane offset plus an immediate below 64 KiB
  const uint32_t ring_lds = __builtin_amdgcn_readfirstlane(lds_addr(ring) + (uint32_t)(tensor * NS * TILE * 2));
  auto issue = [&](int tile, int slot) {
    const uint32_t sbase = ring_lds + (uint32_t)(slot * TILE * 2);
    const int t0 = tile * KT;
    if (t0 + KT <= len) {
      const uint64_t base = uniform64(tb_src + (int64_t)t0 * D);
#pragma unroll
      for (int k = 0; k < PB; ++k) {
        const int rb = (w % WPT) * PB + k;
        const int row = rb * 4 + (lane >> 4);
        const int chunk = (lane & 15) ^ swz16(row);
        dma16_sv(sbase + (uint32_t)(rb * 4 * D * 2), base, (uint32_t)(row * D + chunk * 8) * 2u);
      }
    } else {
      // ragged last tile: rows past the row end repeat its last key (masked)
#pragma unroll
      for (int k = 0; k < PB; ++k) {
        const int rb = (w % WPT) * PB + k;
        const int row = rb * 4 + (lane >> 4);
        const int chunk = (lane & 15) ^ swz16(row);
        const int t = min(t0 + row, len - 1);
        dma16(sbase + (uint32_t)(rb * 4 * D * 2), tb_src + (int64_t)t * D + chunk * 8);
      }
    }
  };

  // prologue: tiles 0 .. 2 in flight before the queries load
  // (the V waves run one tile behind the K waves, as in the loop)
  issue(0, 0);
  if (ntiles > 1) issue(1, 1);
  if (ntiles > 2 && tensor == 0) issue(2, 2);

  // queries of this lane's column n of each query block, rotated, as MFMA B
  // operands: feature 16 kk + 8 g + e; the rotation partner of kk < NKK/2 is
  // chunk kk + NKK/2 of the same lane
  bf16x8_t qb[NKK];
  {
    const int j = min(qbase + n, len - 1);
    const uint16_t* qp = a.q + (((int64_t)it.row * a.W + it.off + j) * a.Hq + h) * D;
    v4u x[NKK];
#pragma unroll
    for (int kk = 0; kk < NKK; ++kk) x[kk] = ld16(qp + 16 * kk + 8 * g);
    if (a.rope) {
#pragma unroll
      for (int kk = 0; kk < NKK / 2; ++kk) rope8(x[kk], x[kk + NKK / 2], 16 * kk + 8 * g, (float)j, a.nl2b);
    }
#pragma unroll
    for (int kk = 0; kk < NKK; ++kk) qb[kk] = __builtin_bit_cast(bf16x8_t, x[kk]);
  }

  // loop-invariant LDS byte offsets of this lane's K and V fragments (V rows
  // 16 apart have the same swizzle, so the K-step ks is a constant offset)
  int koff[NKK];
#pragma unroll
  for (int kk = 0; kk < NKK; ++kk) koff[kk] = (n * D + (((2 * kk + g) ^ swz16(n)) * 8)) * 2;
  const int q16 = lane >> 4, j16 = lane & 15;
  const int vrow = 4 * (q16 >> 1) + (j16 >> 2);
  int voff[NDT][2];
#pragma unroll
  for (int dt = 0; dt < NDT; ++dt)
#pragma unroll
    for (int h2 = 0; h2 < 2; ++h2) {
      const int row = 8 * h2 + vrow;
      const int col = 32 * dt + 16 * (q16 & 1) + 4 * (j16 & 3);
      voff[dt][h2] = (NS * TILE + row * D + (((col >> 3) ^ swz16(row)) * 8) + (col & 7)) * 2;
    }

  f32x16_t o[NDT];
#pragma unroll
  for (int dt = 0; dt < NDT; ++dt)
#pragma unroll
    for (int rr = 0; rr < 16; ++rr) o[dt][rr] = 0.0f;
  float mrun = -__builtin_inff(), mtop = -__builtin_inff(), lsum = 0.0f, alpha = 1.0f;   // mtop = mrun + 8

  // operand fragments of the K and V tiles in a slot (i = 4 ks + dt)
  auto kfrag = [&](int slot, int kk) {
    return *reinterpret_cast<const bf16x8_t*>(reinterpret_cast<const char*>(ring) + koff[kk] + slot * TILE * 2);
  };
  auto vfrag = [&](int slot, int i) {
    const char* vs = reinterpret_cast<const char*>(ring) + slot * TILE * 2 + (i >> 2) * 16 * D * 2;
    const bf16x4_t lo = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_bf16x4*)(vs + voff[i & 3][0]));
    const bf16x4_t hi = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_bf16x4*)(vs + voff[i & 3][1]));
    return (bf16x8_t)__builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
  };
  auto rescale = [&]() {
#pragma unroll
    for (int dt = 0; dt < NDT; ++dt)
#pragma unroll
      for (int rr = 0; rr < 16; ++rr) o[dt][rr] *= alpha;
  };
  // x is computed here: keeps the compiler from sinking it past a fence
  auto pin = [](float& x) { asm volatile("" : "+v"(x)); };
  auto barrier = [] {
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
  };

  // K tile 0 landed (K tiles 1 and 2 may still be in flight), visible to all
  // waves; the loop waits for V
  if (tensor == 0) {
    if (ntiles > 2)
      wait_vm_c<2 * PB>();
    else if (ntiles > 1)
      wait_vm_c<PB>();
    else
      wait_vm_c<0>();
  }
  barrier();

  // two sets of score registers, used in turn by the two halves of each loop
  // trip; one set of probabilities
  f32x16_t sA, sB;
  bf16x8_t pp[2];
  bf16x8_t fr[4];                                    // operand fragments read three MFMAs ahead
  if (active) {
#pragma unroll
    for (int rr = 0; rr < 16; ++rr) sA[rr] = 0.0f;
#pragma unroll
    for (int kk = 0; kk < NKK; ++kk) sA = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kfrag(0, kk), qb[kk], sA, 0, 0, 0);
  }

  // one sub-tile u in ring slot S = u % NS (compile time in the unrolled loop,
  // where every LDS address is then an immediate): sc holds its scores, pp the
  // probabilities of u - 1; writes the scores of u + 1 to sn and the
  // probabilities of u to pp. Sixteen slots of one MFMA each, in an order fixed
  // by scheduling fences: P V of u - 1 (nothing for the first sub-tile), then
  // the scores of u + 1 (of stale LDS contents and discarded for the last);
  // beside them the max, the exponentials, their conversion and sum. Every
  // MFMA's LDS operand is read three MFMAs before it.
  auto sub_tile = [&](auto slot, auto first_tag, int u, f32x16_t& sc, f32x16_t& sn) {
    constexpr bool FIRST = decltype(first_tag)::value;
    const int S = slot, vprev = (slot + NS - 1) % NS, knext = (slot + 1) % NS;
    // K tile u + 1 and V tile u have landed once only one later tile of each
    // (if issued) is in flight. Past the barrier every wave is done with K of
    // u - 1 .. u and V of u - 2, whose slots take K of u + 3 and V of u + 2.
    static_assert(NS == 4 && SPT == 1, "K of u + 3 refills the slot of u - 1, V of u + 2 that of u - 2");
    if (tensor == 0 ? u + 2 < ntiles : u + 1 < ntiles)
      wait_vm_c<PB>();
    else
      wait_vm_c<0>();
    barrier();
    if (tensor == 0) {
      if (u + 3 < ntiles) issue(u + 3, (slot + 3) % NS);
    } else {
      if (u + 2 < ntiles) issue(u + 2, (slot + 2) % NS);
    }
    if (!active) return;
    const int k0 = u * 32;
    if (k0 + 32 > len) {                               // ragged last sub-tile
#pragma unroll
      for (int rr = 0; rr < 16; ++rr) {
        const int key = k0 + 8 * (rr >> 2) + 4 * g + (rr & 3);
        if (key >= len) sc[rr] = -__builtin_inff();
      }
    }
    float m3[4];
    float mx = 0.0f;
    bool resc = false;
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      const int j = i + 3;
      if (j >= 16)
        fr[j & 3] = vfrag(S, j - 16);
      else if (j >= 8)
        fr[j & 3] = kfrag(knext, j - 8);
      else if constexpr (!FIRST)
        fr[j & 3] = vfrag(vprev, j);
      if (i < 8) {
        if constexpr (!FIRST)
          o[i & 3] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fr[i & 3], pp[i >> 2], o[i & 3], 0, 0, 0);
      } else {
        if (i == 8) {
#pragma unroll
          for (int rr = 0; rr < 16; ++rr) sn[rr] = 0.0f;
        }
        sn = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fr[i & 3], qb[i - 8], sn, 0, 0, 0);
      }
      if (i == 1) {
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          m3[r] = vmax(vmax(sc[3 * r], sc[3 * r + 1]), sc[3 * r + 2]);
          pin(m3[r]);
        }
      } else if (i == 2) {
        m3[0] = vmax(vmax(sc[12], sc[13]), m3[0]);
        m3[1] = vmax(vmax(sc[14], sc[15]), m3[1]);
        m3[0] = vmax(vmax(m3[0], m3[1]), m3[2]);
        mx = vmax(m3[0], m3[3]) * a.scale_log2e;       // log2 units
        pin(mx);
      } else if (i == 3) {
        // lazily raised running max: the reference moves only when a score
        // exceeds it by 2^8, so this branch is taken a handful of times per
        // row; the other half-wave holds the other 16 keys of each query
        resc = __builtin_amdgcn_ballot_w64(mx > mtop) != 0;
        if (resc) {
          const auto sw = __builtin_amdgcn_permlane32_swap(__float_as_uint(mx), __float_as_uint(mx), false, false);
          const float mnew = fmaxf(mrun, vmax(__uint_as_float(sw[0]), __uint_as_float(sw[1])));
          alpha = __builtin_amdgcn_exp2f(mrun - mnew);
          lsum *= alpha;
          mrun = mnew;
          mtop = mnew + 8.0f;
        }
      } else if (i >= 4 && i < 12) {
        const int e = 2 * (i - 4);
        float y0 = __builtin_amdgcn_exp2f(fmaf(sc[e], a.scale_log2e, -mrun));
        float y1 = __builtin_amdgcn_exp2f(fmaf(sc[e + 1], a.scale_log2e, -mrun));
        pin(y0);
        pin(y1);
        sc[e] = y0;
        sc[e + 1] = y1;
      }
      if (i >= 5 && i < 13) {
        // P V has read this half of the old probabilities by now
        const int e = 2 * (i - 5);
        pp[e >> 3][e & 7] = (__bf16)sc[e];
        pp[e >> 3][(e & 7) + 1] = (__bf16)sc[e + 1];
      }
      if (i == 9 || i == 13) {
        lsum = add_weights(lsum, pp[i == 9 ? 0 : 1]);
        pin(lsum);
      }
      __builtin_amdgcn_sched_barrier(0);
      if (!FIRST && i == 7 && resc) rescale();         // after P V of u - 1, before that of u
    }
  };

  // u = 0, then four sub-tiles per trip with compile-time slots, then the rest
  sub_tile(Const<0>{}, Const<1>{}, 0, sA, sB);
  int u = 1;
  for (; u + 3 < nsub; u += 4) {
    sub_tile(Const<1>{}, Const<0>{}, u, sB, sA);
    sub_tile(Const<2>{}, Const<0>{}, u + 1, sA, sB);
    sub_tile(Const<3>{}, Const<0>{}, u + 2, sB, sA);
    sub_tile(Const<0>{}, Const<0>{}, u + 3, sA, sB);
  }
  int slot = 1;
  for (; u + 1 < nsub; u += 2, slot += 2) {
    sub_tile(slot, Const<0>{}, u, sB, sA);
    sub_tile(slot + 1, Const<0>{}, u + 1, sA, sB);
  }
  if (u < nsub) sub_tile(slot, Const<0>{}, u, sB, sA);
  if (!active) return;
  {
    const int vs = (nsub - 1) % NS;                    // its first three fragments are read already
#pragma unroll
    for (int i = 0; i < 8; ++i)
      o[i & 3] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(i < 3 ? fr[i] : vfrag(vs, i), pp[i >> 2], o[i & 3], 0, 0, 0);
  }

  // lane (g, n): O^T[feature 32 dt + 8 (rr / 4) + 4 g + rr % 4][query n]
  typedef uint32_t v2u __attribute__((ext_vector_type(2)));
  {
    const int j = qbase + n;
    const float lt = lsum + __shfl_xor(lsum, 32, 64);
    if (j < len) {
      const float inv = 1.0f / lt;
      uint16_t* op = a.out + (((int64_t)it.row * a.W + it.off + j) * a.Hq + h) * D;
#pragma unroll
      for (int dt = 0; dt < NDT; ++dt)
#pragma unroll
        for (int rq = 0; rq < 4; ++rq) {
          const uint32_t w0 = pack_bf16(o[dt][4 * rq + 0] * inv, o[dt][4 * rq + 1] * inv);
          const uint32_t w1 = pack_bf16(o[dt][4 * rq + 2] * inv, o[dt][4 * rq + 3] * inv);
          *reinterpret_cast<v2u*>(op + dt * 32 + 8 * rq + 4 * g) = v2u{w0, w1};
        }
    }
  }
}

}  // namespace

hipError_t launch_refresh_kv(const RefKvArgs& a, int n, int max_len, hipStream_t s) {
  constexpr int D = 128;
  const int64_t units = (int64_t)max_len * a.Hkv * (D / 16);
  const dim3 grid((unsigned)((units + 255) / 256), (unsigned)n);
  hipLaunchKernelGGL(k_refresh_kv<D>, grid, dim3(256), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_refresh_attn(const RefArgs& a, int n_items, hipStream_t s) {
  constexpr int NW = kRefQ / 32;
  hipLaunchKernelGGL((k_refresh_attn<128, NW>), dim3((unsigned)n_items), dim3(64 * NW), 0, s, a);
  return hipGetLastError();
}

}  // namespace bs
