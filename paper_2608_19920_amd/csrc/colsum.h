// The column-sum reduce, shared by its own kernel and by the prefill kernels'
// reduce of both their partial results.
#pragma once

#include "internal.h"

namespace h2o {

constexpr int kColsumThreads = 256;

struct ColsumArgs {
  const float* parts;
  float *wsum, *scores, *copy;
  int nparts, rows_per_part, BH, Nk, ld, G, T, M, Tk;
};
inline ColsumArgs colsum_args(const Shape& s, const Plan& p, const float* parts, float* wsum,
                              ScoreAcc acc) {
  return ColsumArgs{parts, wsum, acc.scores, acc.scores ? acc.copy : nullptr, p.nparts,
                    p.rows_per_part, s.BH(), s.Nk(), p.parts_ld, s.G(), s.T, s.M, s.Tk()};
}

// Block bx of head bh, one column per thread:
// wsum[bh][j] = sum over the partial slots p (in increasing p, so the result
// is bitwise reproducible) whose rows can see column j. With scores
// non-null, a chunk step's accumulation in the same pass: scores[bh][j] +=
// wsum[bh][j] for j < M, one float32 addition of the stored value (the bits
// of the separate accumulate kernel); with copy non-null the sum is also
// written to copy[bh][j], the ranking input of the fused selection.
__device__ __forceinline__ void colsum_reduce_block(const ColsumArgs& a, int bx, int bh) {
  const int j = bx * kColsumThreads + threadIdx.x;
  if (j >= a.Nk) return;
  // the score is requested with the partials, not after them
  float* sc = a.scores && j < a.M ? a.scores + (size_t)bh * a.M + j : nullptr;
  const float s_old = sc ? *sc : 0.f;
  // The partials that see column j are p0 .. nparts-1 (kv_end grows with
  // p): all of them for a cache column, and for chunk key i = j - M those
  // whose last row (r1 - 1) / G reaches i, i.e. (p + 1) * rows_per_part > i * G.
  int p = 0;
  if (a.Tk > 0 && j >= a.M) p = ((j - a.M) * a.G) / a.rows_per_part;
  const float* src = a.parts + ((size_t)p * a.BH + bh) * a.ld + j;
  const size_t stride = (size_t)a.BH * a.ld;
  float s = 0.f;
  // sixteen loads in flight, additions in increasing p (bitwise reproducible)
  for (; p + 15 < a.nparts; p += 16, src += 16 * stride) {
    float v[16];
#pragma unroll
    for (int e = 0; e < 16; ++e) v[e] = src[e * stride];
#pragma unroll
    for (int e = 0; e < 16; ++e) s += v[e];
  }
  for (; p + 3 < a.nparts; p += 4, src += 4 * stride) {
    const float v0 = src[0], v1 = src[stride], v2 = src[2 * stride], v3 = src[3 * stride];
    s += v0;
    s += v1;
    s += v2;
    s += v3;
  }
  for (; p < a.nparts; ++p, src += stride) s += src[0];
  a.wsum[(size_t)bh * a.Nk + j] = s;
  if (sc) {
    const float acc = s_old + s;
    *sc = acc;
    if (a.copy) a.copy[(size_t)bh * a.M + j] = acc;
  }
}

}  // namespace h2o
