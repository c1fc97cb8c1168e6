// Float32 attention of a chunk, forward and backward, on the float32 matrix
// cores (gfx950): v_mfma_f32_16x16x4_f32, float32 operands and accumulators.
//
//   A: lane l holds row l%16, k = l/16        (1 float)
//   B: lane l holds column l%16, k = l/16     (1 float)
//   C: lane l holds rows 4*(l/16) .. +3 of column l%16 (4 floats)
//
// A block owns a few rows (forward, dq: 16 or 32 packed query rows; dk/dv: 16
// keys) and its 8 or 16 waves share out the other side in steps of 16 (wave w
// takes steps w, w + 8, ...), so no wave waits for another inside the loops. What
// all waves use (the block's own rows) sits in LDS; the other side streams
// from global memory straight into operand registers: lane (i, g) reads the
// 16-byte pieces 16t + 4g of row i, and element u of piece t feeds the product
// over the 4 indices 16t + 4g + u. Of a second operand, whose contraction runs
// over the 16 streamed rows, lane (i, g) reads columns 64h + 4i .. +3 of row
// 4g + r: the row that the C layout of the scores holds in register r, so the
// probabilities are an operand as they stand. The waves' partial results meet
// in LDS in a fixed order.
//
// What bounds it: the matrix cores (32 cycles per 16x16x4 product; a step of
// 16 keys and 16 rows is 2 d/4 products forward, against 4 exponentials per
// lane), so probabilities take the full-accuracy expf. At B1 Hq16 Hkv4 d64
// M2048 T256 the attention takes 60 us, dq 57 and dk/dv 76 us, with the matrix
// cores busy 33 to 46 % of the time (operand reads through L1 and a grid of 1 to 2.25
// blocks per CU take the rest); the scalar kernels of sdpa_generic.hip and
// backward.hip take 5,010, 818 and 835 us.
#include "internal.h"

namespace h2o {
namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int kW = 8;            // waves per block (some kernels: twice as many)
constexpr int kStep = 16;        // streamed rows (keys or query rows) per wave step

__device__ __forceinline__ f32x4 mfma(float a, float b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ f32x4 load4(const float* p) {
  return *reinterpret_cast<const f32x4*>(p);
}
// floats per LDS row: 16-byte pieces of 8 consecutive rows fall on distinct banks
template <int D>
__host__ __device__ constexpr int pitch() { return D + 4; }

struct Args {
  const float *q, *kc, *vc, *kn, *vn;
  int Hq, Hkv, G, T, M, Tk, R, Nk;
  KeyPos kp;      // cache mode: token positions
  float scale;
};

__device__ __forceinline__ const float* key_row(const float* cache, const float* fresh,
                                                const Args& a, size_t bh, int j, int D) {
  return j < a.M ? cache + (bh * a.M + j) * (size_t)D
                 : fresh + (bh * a.T + (j - a.M)) * (size_t)D;
}
// Packed row r of KV head (b, h) as a row of [B, Hq, T, .].
__device__ __forceinline__ size_t row_index(const Args& a, int b, int h, int r) {
  return (size_t)(b * a.Hq + h * a.G + r % a.G) * a.T + r / a.G;
}
// Packed row r as (chunk position i, query head g of the group), stepped
// without a division: a lane's rows advance by the same count every step.
struct RowPos {
  int r, i, g;
  __device__ __forceinline__ RowPos(const Args& a, int r0) : r(r0), i(r0 / a.G), g(r0 % a.G) {}
  __device__ __forceinline__ void advance(const Args& a, int n, int ni, int ng) {
    r += n;
    i += ni;
    g += ng;
    if (g >= a.G) { g -= a.G; ++i; }
  }
  // its row of the group's [G, T, .] (row 0 where it lies past R); the group's
  // floats are fewer than 2^30 a head, their bytes a 32-bit offset
  __device__ __forceinline__ uint32_t index(const Args& a) const {
    const bool ok = r < a.R;
    return (uint32_t)((ok ? g : 0) * a.T + (ok ? i : 0));
  }
};
// Earliest chunk position that sees key j (T: none).
template <bool CACHE>
__device__ __forceinline__ int key_rel(const Args& a, size_t bh, int j) {
  if (j >= a.Nk) return a.T;
  if (!CACHE) return j < a.M ? -1 : j - a.M;
  const long long r = (long long)a.kp.tp[bh * a.M + j] - a.kp.pos0;
  return r < -1 ? -1 : (r > a.T ? a.T : (int)r);
}

// Blocks reach the 8 XCDs round-robin: where the heads divide evenly over
// them, a head's blocks go to one XCD and share its L2. x runs last to first
// (later rows see more keys).
__device__ __forceinline__ void block_coords(int& x, int& bh) {
  constexpr int kXcds = 8;
  const int nx = gridDim.x, lin = blockIdx.x + blockIdx.y * gridDim.x;
  if (gridDim.y % kXcds == 0) {
    const int i = lin / kXcds;
    bh = (i / nx) * kXcds + lin % kXcds;
    x = nx - 1 - i % nx;
  } else {
    bh = blockIdx.y;
    x = nx - 1 - blockIdx.x;
  }
}

// Rows [r0, r0 + n) of src (packed query rows of head (b, h)) times mul into
// LDS; rows past R are 0.
template <int D>
__device__ __forceinline__ void stage_rows(float* dst, const float* src, const Args& a, int b,
                                           int h, int r0, int n, float mul) {
  for (int e = threadIdx.x; e < n * (D / 4); e += blockDim.x) {
    const int row = e / (D / 4), c = 4 * (e % (D / 4)), r = r0 + row;
    f32x4 v = {0.f, 0.f, 0.f, 0.f};
    if (r < a.R) v = load4(src + row_index(a, b, h, r) * D + c) * mul;
    *reinterpret_cast<f32x4*>(&dst[row * pitch<D>() + c]) = v;
  }
}

// Operand with k along the streamed row: this lane's pieces of row p.
template <int D>
__device__ __forceinline__ void load_pieces(f32x4 (&v)[D / 16], const float* p, int g4) {
#pragma unroll
  for (int t = 0; t < D / 16; ++t) v[t] = load4(p + 16 * t + 4 * g4);
}

// acc[n] (16 streamed rows x 16 LDS rows 16n ..) += streamed . LDS rows
template <int D, int N>
__device__ __forceinline__ void dot_rows(f32x4 (&acc)[N], const f32x4 (&v)[D / 16],
                                         const float* lds, int l16, int g4) {
#pragma unroll
  for (int n = 0; n < N; ++n) acc[n] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int t = 0; t < D / 16; ++t)
#pragma unroll
    for (int n = 0; n < N; ++n) {
      const f32x4 w = load4(&lds[(16 * n + l16) * pitch<D>() + 16 * t + 4 * g4]);
#pragma unroll
      for (int u = 0; u < 4; ++u) acc[n] = mfma(v[t][u], w[u], acc[n]);
    }
}

// acc[h][u]: element r' of the C block is output column 64h + 4 (4g + r') + u
// of the LDS row (lane's l16); += (streamed rows 4g + r)^T weights[r].
template <int D>
__device__ __forceinline__ void add_rows(f32x4 (&acc)[D / 64][4], const f32x4 (&v)[D / 64][4],
                                         const f32x4& w) {
#pragma unroll
  for (int h = 0; h < D / 64; ++h)
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
      for (int u = 0; u < 4; ++u) acc[h][u] = mfma(v[h][r][u], w[r], acc[h][u]);
}
template <int D>
__device__ __forceinline__ void zero(f32x4 (&acc)[D / 64][4]) {
#pragma unroll
  for (int h = 0; h < D / 64; ++h)
#pragma unroll
    for (int u = 0; u < 4; ++u) acc[h][u] = f32x4{0.f, 0.f, 0.f, 0.f};
}

// A product takes all 16 streamed rows for all 16 LDS rows: a pair that does not
// see each other enters it with weight 0, and 0 times an Inf or NaN is NaN. A
// wave whose sums are not all finite after its loop takes them again with
// add_seen_rows, which leaves such pairs out. Tested inside the loop it took 24
// registers and a block per CU; behind it, B1 Hq16 Hkv4 d64 M2048 T256 takes 59.7,
// 56.7 and 75.8 us (attention, dq, dk/dv) against 58.9, 56.3 and 74.9 without.
// What the second loop is computed from goes through opaque(), so that nothing
// of it is shared with, or kept in registers across, the first.
__device__ __forceinline__ int opaque(int x) {
  asm volatile("" : "+v"(x));
  return x;
}
// nan_if_nonfinite: 0, or NaN where an element is Inf or NaN.
template <int D>
__device__ __forceinline__ float nan_if_nonfinite(const f32x4 (&acc)[D / 64][4]) {
  float z = 0.f;
#pragma unroll
  for (int h = 0; h < D / 64; ++h)
#pragma unroll
    for (int u = 0; u < 4; ++u)
#pragma unroll
      for (int r = 0; r < 4; ++r) z = fmaf(acc[h][u][r], 0.f, z);
  return z;
}
// add_rows over the pairs that see each other: the streamed rows one by one, row(k)
// their address. hidden: bit r set where this lane's pair of row 4 g4 + r is hidden.
template <int D, class Row>
__device__ __forceinline__ void add_seen_rows(f32x4 (&acc)[D / 64][4], const f32x4& w, int hidden,
                                              int l16, int g4, Row&& row) {
#pragma unroll 1
  for (int k = 0; k < kStep; ++k) {
    const int from = 16 * (k >> 2) + l16, r = k & 3;
    const float wr = r == 0 ? w[0] : r == 1 ? w[1] : r == 2 ? w[2] : w[3];
    const float p = __shfl(wr, from, 64);
    const bool seen = !((__shfl(hidden, from, 64) >> r) & 1);
    const float* src = row(k) + 16 * g4;
#pragma unroll
    for (int h = 0; h < D / 64; ++h)
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        const f32x4 x = load4(src + 64 * h + 4 * c);
#pragma unroll
        for (int u = 0; u < 4; ++u) acc[h][u][c] = seen ? fmaf(p, x[u], acc[h][u][c]) : acc[h][u][c];
        __builtin_amdgcn_sched_barrier(0);   // few registers: the path is rare
      }
  }
}

// acc of all waves added into wave 0's, in a fixed tree order, through LDS of
// NW/2 x n x 16 rows of pitch<D>() floats. Every thread of the block calls it.
template <int D, int N, int NW>
__device__ __forceinline__ void reduce_waves(f32x4 (&acc)[N][D / 64][4], float* red, int wave,
                                             int l16, int g4) {
  constexpr int P = pitch<D>();
#pragma unroll
  for (int s = NW / 2; s >= 1; s >>= 1) {
    __syncthreads();
    if (wave >= s && wave < 2 * s) {
      float* dst = red + (size_t)(wave - s) * N * 16 * P;
#pragma unroll
      for (int n = 0; n < N; ++n)
#pragma unroll
        for (int h = 0; h < D / 64; ++h)
#pragma unroll
          for (int u = 0; u < 4; ++u)
            *reinterpret_cast<f32x4*>(&dst[(16 * n + l16) * P + 64 * h + 16 * u + 4 * g4]) =
                acc[n][h][u];
    }
    __syncthreads();
    if (wave < s) {
      const float* src = red + (size_t)wave * N * 16 * P;
#pragma unroll
      for (int n = 0; n < N; ++n)
#pragma unroll
        for (int h = 0; h < D / 64; ++h)
#pragma unroll
          for (int u = 0; u < 4; ++u)
            acc[n][h][u] += load4(&src[(16 * n + l16) * P + 64 * h + 16 * u + 4 * g4]);
    }
  }
}
// One lane's share of an output row: 4 consecutive columns per (h, r).
template <int D>
__device__ __forceinline__ void store_row(float* dst, const f32x4 (&acc)[D / 64][4], int g4,
                                          float mul) {
#pragma unroll
  for (int h = 0; h < D / 64; ++h)
#pragma unroll
    for (int r = 0; r < 4; ++r)
      *reinterpret_cast<f32x4*>(dst + 64 * h + 16 * g4 + 4 * r) =
          f32x4{acc[h][0][r], acc[h][1][r], acc[h][2][r], acc[h][3][r]} * mul;
}

// Sum of v over the 16 lanes of a DPP row, in every lane.
__device__ __forceinline__ float row16_sum(float v) {
#pragma unroll
  for (int o = 1; o < 16; o <<= 1) v += __shfl_xor(v, o, 64);
  return v;
}

// ------------------------------------------------------------------ forward
// 16 NQB packed rows per block: a sweep over the keys for each row's maximum
// and sum, merged over the waves to lambda; a second sweep with the exact
// probabilities for the output and the block's column sums (a wave alone
// holds a key's probabilities, so it stores their sum over the rows itself).
template <int D, int NQB, bool CACHE, int NW>
__global__ __launch_bounds__(NW * 64) void f32_attend(Args a, float* __restrict__ out,
                                                  float* __restrict__ lse,
                                                  float* __restrict__ parts) {
  constexpr int ROWS = 16 * NQB, P = pitch<D>();
  __shared__ __attribute__((aligned(16))) float Qs[ROWS * P];
  __shared__ __attribute__((aligned(16))) float red[NW / 2 * ROWS * P];
  __shared__ float2 st[NW][ROWS];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int l16 = lane & 15, g4 = lane >> 4;
  int x, bhi;
  block_coords(x, bhi);
  const size_t bh = bhi;
  const int b = bhi / a.Hkv, h = bhi % a.Hkv, row0 = x * ROWS;
  stage_rows<D>(Qs, a.q, a, b, h, row0, ROWS, a.scale);
  __syncthreads();
  const int kv_end = kv_end_for_rows(min(row0 + ROWS, a.R), a.G, a.T, a.M, a.Tk);
  const int nsteps = (kv_end + kStep - 1) / kStep;
  int qi[NQB];
  float m[NQB], l[NQB];
#pragma unroll
  for (int n = 0; n < NQB; ++n) {
    qi[n] = (row0 + 16 * n + l16) / a.G;
    m[n] = -INFINITY;
    l[n] = 0.f;
  }
  f32x4 k0[D / 16], k1[D / 16];
  auto load_k = [&](f32x4 (&k)[D / 16], int s) {
    const int j = min(s * kStep + l16, kv_end - 1);
    load_pieces<D>(k, key_row(a.kc, a.kn, a, bh, j, D), g4);
  };
  auto rel_of = [&](int (&rel)[4], int s) {
#pragma unroll
    for (int r = 0; r < 4; ++r) rel[r] = key_rel<CACHE>(a, bh, s * kStep + 4 * g4 + r);
  };
  if (wave < nsteps) load_k(k0, wave);
  for (int s = wave; s < nsteps; s += NW) {
    if (s + NW < nsteps) load_k(k1, s + NW);
    int rel[4];
    rel_of(rel, s);
    f32x4 sc[NQB];
    dot_rows<D, NQB>(sc, k0, Qs, l16, g4);
#pragma unroll
    for (int n = 0; n < NQB; ++n) {
      float mn = m[n];
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        if (rel[r] > qi[n]) sc[n][r] = -INFINITY;
        mn = fmaxf(mn, sc[n][r]);
      }
      const float ref = mn == -INFINITY ? 0.f : mn;
      float t = l[n] * expf(m[n] - ref);
#pragma unroll
      for (int r = 0; r < 4; ++r) t += expf(sc[n][r] - ref);
      l[n] = t;
      m[n] = mn;
    }
#pragma unroll
    for (int t = 0; t < D / 16; ++t) k0[t] = k1[t];
  }
  if (wave < nsteps) load_k(k0, wave);   // for the second sweep
  // merge the lane groups (disjoint keys of one row), then the waves
  auto merge = [](float& m1, float& l1, float m2, float l2) {
    const float mn = fmaxf(m1, m2), ref = mn == -INFINITY ? 0.f : mn;
    l1 = l1 * expf(m1 - ref) + l2 * expf(m2 - ref);
    m1 = mn;
  };
#pragma unroll
  for (int n = 0; n < NQB; ++n) {
#pragma unroll
    for (int o = 16; o <= 32; o <<= 1)
      merge(m[n], l[n], __shfl_xor(m[n], o, 64), __shfl_xor(l[n], o, 64));
    if (g4 == 0) st[wave][16 * n + l16] = make_float2(m[n], l[n]);
  }
  __syncthreads();
  float lam[NQB];
#pragma unroll
  for (int n = 0; n < NQB; ++n) {
    float2 v = st[0][16 * n + l16];
#pragma unroll
    for (int w = 1; w < NW; ++w) {
      const float2 y = st[w][16 * n + l16];
      merge(v.x, v.y, y.x, y.y);
    }
    const int r = row0 + 16 * n + l16;
    const float lm = v.y == 0.f ? -INFINITY : v.x + logf(v.y);   // a NaN stays one
    if (wave == 0 && g4 == 0 && r < a.R) lse[row_index(a, b, h, r)] = lm;
    lam[n] = lm;
    // no key seen, or a padding row: no key is visible to it
    if (r >= a.R || lm == -INFINITY) qi[n] = INT32_MIN;
  }

  f32x4 o[NQB][D / 64][4];
#pragma unroll
  for (int n = 0; n < NQB; ++n) zero<D>(o[n]);
  float* prow = parts + ((size_t)x * gridDim.y + bh) * a.Nk;
  for (int s = wave; s < nsteps; s += NW) {
    f32x4 v[D / 64][4];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int j = min(s * kStep + 4 * g4 + r, kv_end - 1);
      const float* p = key_row(a.vc, a.vn, a, bh, j, D) + 4 * l16;
#pragma unroll
      for (int hh = 0; hh < D / 64; ++hh) v[hh][r] = load4(p + 64 * hh);
    }
    int rel[4];
    rel_of(rel, s);
    f32x4 sc[NQB];
    dot_rows<D, NQB>(sc, k0, Qs, l16, g4);
    // the next keys into the registers just read, behind the output products
    __builtin_amdgcn_sched_barrier(0);
    if (s + NW < nsteps) load_k(k0, s + NW);
    f32x4 cs = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int n = 0; n < NQB; ++n) {
#pragma unroll
      for (int r = 0; r < 4; ++r) sc[n][r] = rel[r] > qi[n] ? 0.f : expf(sc[n][r] - lam[n]);
      cs += sc[n];
    }
#pragma unroll
    for (int n = 0; n < NQB; ++n) add_rows<D>(o[n], v, sc[n]);
#pragma unroll
    for (int r = 0; r < 4; ++r) cs[r] = row16_sum(cs[r]);
    const int j = s * kStep + 4 * g4 + l16;
    if (l16 < 4 && j < kv_end)
      prow[j] = l16 == 0 ? cs[0] : l16 == 1 ? cs[1] : l16 == 2 ? cs[2] : cs[3];
  }
  float z = 0.f;
#pragma unroll
  for (int n = 0; n < NQB; ++n) z += nan_if_nonfinite<D>(o[n]);
  if (__builtin_expect(__builtin_amdgcn_ballot_w64(z != 0.f) != 0, 0)) {   // wave-uniform
    const int wv = __builtin_amdgcn_readfirstlane(opaque(wave)), li = opaque(l16), gi = opaque(g4);
#pragma unroll
    for (int n = 0; n < NQB; ++n) zero<D>(o[n]);
#pragma unroll 1
    for (int s = wv; s < nsteps; s += NW) {
      f32x4 k[D / 16], sc[NQB];
      load_pieces<D>(k, key_row(a.kc, a.kn, a, bh, min(s * kStep + li, kv_end - 1), D), gi);
      dot_rows<D, NQB>(sc, k, Qs, li, gi);
#pragma unroll
      for (int n = 0; n < NQB; ++n) {
        int hidden = 0;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          hidden |= (int)(key_rel<CACHE>(a, bh, s * kStep + 4 * gi + r) > qi[n]) << r;
          sc[n][r] = expf(sc[n][r] - lam[n]);
        }
        add_seen_rows<D>(o[n], sc[n], hidden, li, gi, [&](int i) {
          return key_row(a.vc, a.vn, a, bh, min(s * kStep + i, kv_end - 1), D);
        });
      }
    }
  }
  reduce_waves<D, NQB, NW>(o, red, wave, l16, g4);
  if (wave == 0) {
#pragma unroll
    for (int n = 0; n < NQB; ++n) {
      const int r = row0 + 16 * n + l16;
      if (r < a.R) store_row<D>(out + row_index(a, b, h, r) * D, o[n], g4, 1.f);
    }
  }
}

// ----------------------------------------------------------------- backward
// dQ_r = scale (sum_j P dP K_j - D_r sum_j P K_j) and D_r = sum_j P dP from
// one sweep over the keys, 16 packed rows per block.
// At d = 128 a block of 8 waves is alone on its CU: told so (two waves per SIMD),
// and with the masks behind the products, the compiler keeps more loads in
// flight (B1 Hq16 Hkv4 M2048 T256 121 -> 110 us).
template <int D, bool CACHE, int NW>
__global__ __launch_bounds__(NW * 64) __attribute__((amdgpu_waves_per_eu(2, D == 64 ? 8 : 2)))
void f32_bwd_dq(Args a, const float* __restrict__ dout, const float* __restrict__ lse,
                float* __restrict__ dq, float* __restrict__ dot) {
  constexpr int P = pitch<D>();
  __shared__ __attribute__((aligned(16))) float Qs[16 * P], Os[16 * P];
  __shared__ __attribute__((aligned(16))) float red[NW / 2 * 16 * P];
  __shared__ float ds[NW][16];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int l16 = lane & 15, g4 = lane >> 4;
  int x, bhi;
  block_coords(x, bhi);
  const size_t bh = bhi;
  const int b = bhi / a.Hkv, h = bhi % a.Hkv, row0 = x * 16;
  stage_rows<D>(Qs, a.q, a, b, h, row0, 16, 1.f);
  stage_rows<D>(Os, dout, a, b, h, row0, 16, 1.f);
  __syncthreads();
  const int kv_end = kv_end_for_rows(min(row0 + 16, a.R), a.G, a.T, a.M, a.Tk);
  const int nsteps = (kv_end + kStep - 1) / kStep;
  const int r = row0 + l16;
  const float lam = r < a.R ? lse[row_index(a, b, h, r)] : -INFINITY;
  const int qi = lam > -INFINITY ? r / a.G : INT32_MIN;   // no key seen: none visible
  f32x4 ad[1][D / 64][4], ap[D / 64][4];
  zero<D>(ad[0]);
  zero<D>(ap);
  float dsum = 0.f;
  for (int s = wave; s < nsteps; s += NW) {
    f32x4 k[D / 16], v[D / 16], kt[D / 64][4];
    const int jr = min(s * kStep + l16, kv_end - 1);
    load_pieces<D>(k, key_row(a.kc, a.kn, a, bh, jr, D), g4);
    load_pieces<D>(v, key_row(a.vc, a.vn, a, bh, jr, D), g4);
    f32x4 sc[1], dp[1];
    dot_rows<D, 1>(sc, k, Qs, l16, g4);
    dot_rows<D, 1>(dp, v, Os, l16, g4);
    int rel[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) rel[u] = key_rel<CACHE>(a, bh, s * kStep + 4 * g4 + u);
    // the second read of k goes out once the first is used (registers)
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int j = min(s * kStep + 4 * g4 + u, kv_end - 1);
      const float* p = key_row(a.kc, a.kn, a, bh, j, D) + 4 * l16;
#pragma unroll
      for (int hh = 0; hh < D / 64; ++hh) kt[hh][u] = load4(p + 64 * hh);
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const float p = rel[u] > qi ? 0.f : expf(sc[0][u] * a.scale - lam);
      sc[0][u] = p;
      dp[0][u] *= p;
      dsum += dp[0][u];
    }
    add_rows<D>(ad[0], kt, dp[0]);
    add_rows<D>(ap, kt, sc[0]);
  }
  const float z = nan_if_nonfinite<D>(ad[0]) + nan_if_nonfinite<D>(ap) + dsum * 0.f;
  if (__builtin_expect(__builtin_amdgcn_ballot_w64(z != 0.f) != 0, 0)) {   // wave-uniform
    const int wv = __builtin_amdgcn_readfirstlane(opaque(wave)), li = opaque(l16), gi = opaque(g4);
    zero<D>(ad[0]);
    zero<D>(ap);
    dsum = 0.f;
#pragma unroll 1
    for (int s = wv; s < nsteps; s += NW) {
      auto key = [&](int k) { return min(s * kStep + k, kv_end - 1); };
      f32x4 v[D / 16], sc[1], dp[1];
      load_pieces<D>(v, key_row(a.kc, a.kn, a, bh, key(li), D), gi);
      dot_rows<D, 1>(sc, v, Qs, li, gi);
      load_pieces<D>(v, key_row(a.vc, a.vn, a, bh, key(li), D), gi);
      dot_rows<D, 1>(dp, v, Os, li, gi);
      int hidden = 0;
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const bool hid = key_rel<CACHE>(a, bh, s * kStep + 4 * gi + u) > qi;
        hidden |= (int)hid << u;
        sc[0][u] = expf(sc[0][u] * a.scale - lam);
        dp[0][u] *= sc[0][u];
        if (!hid) dsum += dp[0][u];
      }
      auto row = [&](int k) { return key_row(a.kc, a.kn, a, bh, key(k), D); };
      add_seen_rows<D>(ad[0], dp[0], hidden, li, gi, row);
      add_seen_rows<D>(ap, sc[0], hidden, li, gi, row);
    }
  }
  dsum += __shfl_xor(dsum, 16, 64);
  dsum += __shfl_xor(dsum, 32, 64);
  if (g4 == 0) ds[wave][l16] = dsum;
  __syncthreads();
  float d = ds[0][l16];
#pragma unroll
  for (int w = 1; w < NW; ++w) d += ds[w][l16];
#pragma unroll
  for (int hh = 0; hh < D / 64; ++hh)
#pragma unroll
    for (int u = 0; u < 4; ++u) ad[0][hh][u] -= d * ap[hh][u];
  reduce_waves<D, 1, NW>(ad, red, wave, l16, g4);
  if (wave == 0 && r < a.R) {
    store_row<D>(dq + row_index(a, b, h, r) * D, ad[0], g4, a.scale);
    if (g4 == 0) dot[bh * a.R + r] = d;
  }
}

// dV_j = sum_r P_rj dout_r and dK_j = scale sum_r P (dP - D_r) Q_r over the
// head's packed rows, 16 keys per block. 128 registers at d = 64 (two blocks per CU);
// the group's rows are addressed by 32-bit offsets, which keeps the kernels free
// of spills.
template <int D, bool CACHE, int NW>
__global__ __launch_bounds__(NW * 64)
__attribute__((amdgpu_waves_per_eu(D == 64 ? 4 : 2, D == 64 ? 4 : 8)))
void f32_bwd_dkdv(Args a, const float* __restrict__ dout, const float* __restrict__ lse,
                  const float* __restrict__ dot, float* __restrict__ dkc,
                  float* __restrict__ dvc, float* __restrict__ dkn, float* __restrict__ dvn) {
  constexpr int P = pitch<D>();
  __shared__ __attribute__((aligned(16))) float Ks[16 * P], Vs[16 * P];
  __shared__ __attribute__((aligned(16))) float red[NW / 2 * 16 * P];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int l16 = lane & 15, g4 = lane >> 4;
  int x, bhi;
  block_coords(x, bhi);
  x = gridDim.x - 1 - x;   // first keys first: they are seen by the most rows
  const size_t bh = bhi;
  const int b = bhi / a.Hkv, h = bhi % a.Hkv, j0 = x * 16;
  for (int e = threadIdx.x; e < 16 * (D / 4); e += NW * 64) {
    const int row = e / (D / 4), c = 4 * (e % (D / 4)), j = min(j0 + row, a.Nk - 1);
    *reinterpret_cast<f32x4*>(&Ks[row * P + c]) = load4(key_row(a.kc, a.kn, a, bh, j, D) + c);
    *reinterpret_cast<f32x4*>(&Vs[row * P + c]) = load4(key_row(a.vc, a.vn, a, bh, j, D) + c);
  }
  __syncthreads();
  const int j = j0 + l16;
  const int rel = key_rel<CACHE>(a, bh, j);
  // rows before the block's first chunk key see none of its keys
  const int s0 = !CACHE && j0 > a.M ? (j0 - a.M) * a.G / kStep : 0;
  const int s1 = (a.R + kStep - 1) / kStep;
  f32x4 dk[1][D / 64][4], dv[1][D / 64][4];
  zero<D>(dk[0]);
  zero<D>(dv[0]);
  constexpr int kAdv = kStep * NW;
  const int ni = kAdv / a.G, ng = kAdv % a.G;
  const size_t group = (size_t)(b * a.Hq + h * a.G) * a.T;
  const float *qh = a.q + group * D, *dh = dout + group * D, *lh = lse + group;
  auto at = [](const float* base, uint32_t bytes) {
    return reinterpret_cast<const float*>(reinterpret_cast<const char*>(base) + bytes);
  };
  RowPos pa(a, (s0 + wave) * kStep + l16), pb(a, (s0 + wave) * kStep + 4 * g4);
  for (int s = s0 + wave; s < s1; s += NW) {
    f32x4 q[D / 16], od[D / 16], qt[D / 64][4], ot[D / 64][4];
    const uint32_t ra = pa.index(a) * (uint32_t)(D * 4);
    load_pieces<D>(q, at(qh, ra), g4);
    load_pieces<D>(od, at(dh, ra), g4);
    float lam[4], dr[4];
    int pos[4];
    uint32_t row[4];   // bytes
    RowPos pu = pb;
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const bool ok = pu.r < a.R;
      const uint32_t ri = pu.index(a);
      row[u] = ri * (uint32_t)(D * 4) + 16u * l16;
      lam[u] = *at(lh, ri * 4u);
      dr[u] = dot[bh * a.R + (ok ? pu.r : 0)];
      pos[u] = ok && lam[u] > -INFINITY ? pu.i : INT32_MIN;   // none visible
#pragma unroll
      for (int hh = 0; hh < D / 64; ++hh)
        ot[hh][u] = load4(at(dh, row[u] + 256u * hh));
      pu.advance(a, 1, 0, 1);
    }
    pa.advance(a, kAdv, ni, ng);
    pb.advance(a, kAdv, ni, ng);
    f32x4 sc[1], dp[1];
    dot_rows<D, 1>(sc, q, Ks, l16, g4);
    dot_rows<D, 1>(dp, od, Vs, l16, g4);
    // the second read of q goes out behind the dV products (registers)
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int u = 0; u < 4; ++u)
#pragma unroll
      for (int hh = 0; hh < D / 64; ++hh)
        qt[hh][u] = load4(at(qh, row[u] + 256u * hh));
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const float p = rel > pos[u] ? 0.f : expf(sc[0][u] * a.scale - lam[u]);
      sc[0][u] = p;
      dp[0][u] = p * (dp[0][u] - dr[u]);
    }
    add_rows<D>(dv[0], ot, sc[0]);
    add_rows<D>(dk[0], qt, dp[0]);
  }
  const float z = nan_if_nonfinite<D>(dk[0]) + nan_if_nonfinite<D>(dv[0]);
  if (__builtin_expect(__builtin_amdgcn_ballot_w64(z != 0.f) != 0, 0)) {   // wave-uniform
    const int wv = __builtin_amdgcn_readfirstlane(opaque(wave)), li = opaque(l16), gi = opaque(g4);
    zero<D>(dk[0]);
    zero<D>(dv[0]);
#pragma unroll 1
    for (int s = s0 + wv; s < s1; s += NW) {
      // packed row s kStep + k as a row of [B, Hq, T, .] (row 0 where it lies past R)
      auto packed = [&](int k) { return s * kStep + k < a.R ? s * kStep + k : 0; };
      f32x4 v[D / 16], sc[1], dp[1];
      load_pieces<D>(v, a.q + row_index(a, b, h, packed(li)) * D, gi);
      dot_rows<D, 1>(sc, v, Ks, li, gi);
      load_pieces<D>(v, dout + row_index(a, b, h, packed(li)) * D, gi);
      dot_rows<D, 1>(dp, v, Vs, li, gi);
      int hidden = 0;
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int r = packed(4 * gi + u);
        const float lam = lse[row_index(a, b, h, r)];
        const bool hid = s * kStep + 4 * gi + u >= a.R || !(lam > -INFINITY) || rel > r / a.G;
        hidden |= (int)hid << u;
        sc[0][u] = expf(sc[0][u] * a.scale - lam);
        dp[0][u] = sc[0][u] * (dp[0][u] - dot[bh * a.R + r]);
      }
      add_seen_rows<D>(dv[0], sc[0], hidden, li, gi, [&](int k) {
        return dout + row_index(a, b, h, packed(k)) * D;
      });
      add_seen_rows<D>(dk[0], dp[0], hidden, li, gi, [&](int k) {
        return a.q + row_index(a, b, h, packed(k)) * D;
      });
    }
  }
  reduce_waves<D, 1, NW>(dk, red, wave, l16, g4);
  reduce_waves<D, 1, NW>(dv, red, wave, l16, g4);
  const int jo = j0 + opaque(l16);   // j, not kept through the loop
  if (wave == 0 && jo < a.Nk) {
    const bool cached = jo < a.M;
    const size_t o = (cached ? bh * a.M + jo : bh * a.T + (jo - a.M)) * (size_t)D;
    store_row<D>((cached ? dkc : dkn) + o, dk[0], g4, a.scale);
    store_row<D>((cached ? dvc : dvn) + o, dv[0], g4, 1.f);
  }
}

Args make_args(const Shape& s, const void* q, const void* kc, const void* vc, const void* kn,
               const void* vn, float scale, KeyPos kp) {
  return Args{(const float*)q, (const float*)kc, (const float*)vc, (const float*)kn,
              (const float*)vn, s.Hq, s.Hkv, s.G(), s.T, s.M, s.Tk(), s.R(), s.Nk(), kp, scale};
}

// Waves per block: 16 for the row kernels that fit 128 registers (d = 64, 16
// rows), so that a grid of one block per CU still has four waves per SIMD
// (59 against 61 us attending and 56 against 59 us for dq, at the size
// above); 8 otherwise (dk/dv: 75 us with 8, 84 with 16).
template <int D, bool CACHE>
hipError_t attend(const Shape& s, const Plan& p, const Args& a, float* out, float* lse, char* ws,
                  hipStream_t st) {
  float* parts = reinterpret_cast<float*>(ws + p.off_parts);
  auto go = [&](auto kern, int waves) {
    return launch_kernel(K_F32_ATTEND, kern, dim3(p.nparts, s.BH()), dim3(64 * waves), st, a, out,
                         lse, parts);
  };
  if (p.rows_per_part == 32) return go(f32_attend<D, 2, CACHE, kW>, kW);
  constexpr int NW = D == 64 ? 2 * kW : kW;
  return go(f32_attend<D, 1, CACHE, NW>, NW);
}

template <int D, bool CACHE>
hipError_t backward(const Shape& s, const Args& a, const float* lse, const float* dout, float* dq,
                    float* dkc, float* dvc, float* dkn, float* dvn, float* dot, hipStream_t st) {
  constexpr int NW = D == 64 ? 2 * kW : kW;
  hipError_t e = launch_kernel(K_BWD_DQ, f32_bwd_dq<D, CACHE, NW>,
                               dim3((s.R() + 15) / 16, s.BH()), dim3(64 * NW), st, a, dout, lse,
                               dq, dot);
  if (e != hipSuccess) return e;
  return launch_kernel(K_BWD_DKDV, f32_bwd_dkdv<D, CACHE, kW>, dim3((s.Nk() + 15) / 16, s.BH()),
                       dim3(64 * kW), st, a, dout, lse, (const float*)dot, dkc, dvc, dkn, dvn);
}

}  // namespace

hipError_t launch_sdpa_f32(const Shape& s, const Plan& p, const void* q, const void* kc,
                           const void* vc, const void* kn, const void* vn, void* out, float* lse,
                           float* wsum, char* ws, float scale, KeyPos kp, hipStream_t st,
                           ScoreAcc acc) {
  const Args a = make_args(s, q, kc, vc, kn, vn, scale, kp);
  const bool cache = kp.tp != nullptr;
  auto go = [&](auto fn) { return fn(s, p, a, (float*)out, lse, ws, st); };
  const hipError_t e = s.d == 64 ? (cache ? go(attend<64, true>) : go(attend<64, false>))
                                 : (cache ? go(attend<128, true>) : go(attend<128, false>));
  if (e != hipSuccess) return e;
  return launch_colsum_reduce(s, p, reinterpret_cast<float*>(ws + p.off_parts), wsum, st, acc);
}

hipError_t launch_sdpa_backward_f32(const Shape& s, const void* q, const void* kc, const void* vc,
                                    const void* kn, const void* vn, KeyPos kp, const float* lse,
                                    const void* dout, void* dq, void* dkc, void* dvc, void* dkn,
                                    void* dvn, float* dot, float scale, hipStream_t st) {
  const Args a = make_args(s, q, kc, vc, kn, vn, scale, kp);
  const bool cache = kp.tp != nullptr;
  auto go = [&](auto fn) {
    return fn(s, a, lse, (const float*)dout, (float*)dq, (float*)dkc, (float*)dvc, (float*)dkn,
              (float*)dvn, dot, st);
  };
  return s.d == 64 ? (cache ? go(backward<64, true>) : go(backward<64, false>))
                   : (cache ? go(backward<128, true>) : go(backward<128, false>));
}

}  // namespace h2o
