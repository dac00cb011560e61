// Split-KV merge (device code shared by the merge launch of the attention and
// by the row reductions of a fused step, which carry it beside their own work).
#pragma once

#include "bs_internal.h"

namespace bs {

// Workgroups of 256 threads of the merge: one wave per split row, wave slot of
// its pieces' workgroups and group of 4 output features.
inline int merge_blocks(const AttnArgs& a) { return (a.n_merge * a.G * a.RBW * (a.D / 8) + 3) / 4; }

// Workgroup b of the merge. Wave (r, wg, k) combines group k (4 of the lane's output
// features) of split row r for wave slot wg of its pieces' workgroups, which
// serve query head kvh * G + wg / RBW and 32 block rows (row block
// rb + wg % RBW). Lane (g, n) folds the pieces' partials of its query column
// with a running max m: the sums so far are scaled by 2^(m_old - m) and piece
// p's by 2^(m_p - m) (the log-sum-exp merge of softmax pieces), eight pieces'
// loads in flight at a time; the quotient is written like the attention's own
// output (bf16; rows B .. L - 1 as zeros). Every load of a wave is one
// contiguous 256 B or 1 KiB run.
//
// Latency bounds it, so a wave takes one group only: with a quarter of the
// groups per wave (the max and sum of a piece read once per wave) the merge of
// 92 rows in 224 pieces took 16.4 us instead of 10.9.
//
// UNIFORM: the row's entry is read through scalar loads and its fields stay in
// SGPRs. That is the faster form while rows have few pieces (calls: 128 rows of 2
// 30.55 -> 29.9 us, 64 rows of 2-4 33.7 -> 33.0, 8 rows of 11 beside 80 of 2: 45.1 ->
// 44.4), and the slower one where some rows take several batches beside many
// that take one (4 rows of 27 beside 36 of 2: 32.9 -> 33.4; the merge itself 9.32
// -> 9.76). Few rows of 15 pieces: the same in both.
template <int D, bool UNIFORM>
__device__ inline void merge_rows(const AttnArgs& a, int b) {
  typedef float f32x4_t __attribute__((ext_vector_type(4)));
  constexpr int NG = D / 8;                       // groups of 4 floats per lane
  constexpr int OFL = NG * 64 * 4;
  constexpr int CH = kMergeBatch;
  const int GW = a.G * a.RBW;
  const int wl = b * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int wv = UNIFORM ? __builtin_amdgcn_readfirstlane(wl) : wl;
  if (wv >= a.n_merge * GW * NG) return;
  const int k = wv % NG, wg = (wv / NG) % GW;
  const AttnMerge mg = a.merges[wv / (NG * GW)];
  const int g = lane >> 5, n = lane & 31;
  const int h = mg.kvh * a.G + wg / a.RBW;
  const int j = (mg.rb + wg % a.RBW) * 32 + n;
  const int64_t pstride = (int64_t)GW * part_wave_floats(D);
  const float* pw = a.parts + ((int64_t)mg.part0 * GW + wg) * part_wave_floats(D);
  f32x4_t acc = f32x4_t{0.0f, 0.0f, 0.0f, 0.0f};
  float m = -__builtin_inff(), l = 0.0f;
  for (int p0 = 0; p0 < mg.nparts; p0 += CH) {
    float mp[CH], lp[CH];
    f32x4_t op[CH];
#pragma unroll
    for (int i = 0; i < CH; ++i) {
      if (p0 + i < mg.nparts) {
        const float* pp = pw + (p0 + i) * pstride;
        mp[i] = pp[OFL + lane];
        lp[i] = pp[OFL + 64 + lane];
        op[i] = *reinterpret_cast<const f32x4_t*>(pp + (k * 64 + lane) * 4);
      } else {
        mp[i] = -__builtin_inff();
        lp[i] = 0.0f;
        op[i] = f32x4_t{0.0f, 0.0f, 0.0f, 0.0f};
      }
    }
    float mn = m;
#pragma unroll
    for (int i = 0; i < CH; ++i) mn = fmaxf(mn, mp[i]);
    const float sa = __builtin_amdgcn_exp2f(m - mn);
    l *= sa;
    acc *= sa;
#pragma unroll
    for (int i = 0; i < CH; ++i) {
      const float sb = __builtin_amdgcn_exp2f(mp[i] - mn);     // 0 for the padding entries
      l = fmaf(lp[i], sb, l);
      acc += op[i] * sb;
    }
    m = mn;
  }
  if (j >= a.L) return;
  const float inv = j < mg.B ? 1.0f / l : 0.0f;
  // group k = 4 dt + rq holds features 32 dt + 8 rq + 4 g .. + 3
  uint16_t* op = static_cast<uint16_t*>(a.out) + (((int64_t)mg.req * a.L + j) * a.Hq + h) * D +
                 32 * (k >> 2) + 8 * (k & 3) + 4 * g;
  typedef uint32_t v2u __attribute__((ext_vector_type(2)));
  uint32_t w2[2];
#pragma unroll
  for (int e = 0; e < 2; ++e) {
    const __bf16 lo = (__bf16)(acc[2 * e] * inv), hi = (__bf16)(acc[2 * e + 1] * inv);
    w2[e] = (uint32_t)__builtin_bit_cast(uint16_t, lo) | ((uint32_t)__builtin_bit_cast(uint16_t, hi) << 16);
  }
  __builtin_nontemporal_store(v2u{w2[0], w2[1]}, reinterpret_cast<v2u*>(op));
}

}  // namespace bs
