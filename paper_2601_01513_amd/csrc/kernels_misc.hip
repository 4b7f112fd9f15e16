// Memory-bound helper kernels of the verifier scoring pass: rotary table,
// per-row tables, embedding gathers, RMSNorm, LM-head inputs, the log-sum-exp
// merge with the target gather, and the per-candidate sum and argmax
// (Eq. 6-7). All of them read and write rows with consecutive lanes on
// consecutive elements; reductions run in a fixed order (no atomics).
#include <algorithm>

#include "common.h"

namespace vsr {

// Sum over a 256-thread block, same value returned to every thread.
__device__ __forceinline__ float block_sum256(float v, float *red) {
  v = wave_sum(v);
  const int w = threadIdx.x >> 6, l = threadIdx.x & 63;
  __syncthreads();
  if (l == 0) red[w] = v;
  __syncthreads();
  return (red[0] + red[1]) + (red[2] + red[3]);
}

// ------------------------------------------------------------- rotary table
__global__ void k_rope_table(float2 *cs, int npos, int hd, double base) {
  const int half = hd / 2;
  const long idx = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= (long)npos * half) return;
  const int p = (int)(idx / half), i = (int)(idx % half);
  const double inv = pow(base, -2.0 * i / hd);
  const double ang = (double)p * inv;
  cs[idx] = make_float2((float)cos(ang), (float)sin(ang));
}

hipError_t launch_rope_table(float2 *cs, int npos, int hd, float base, hipStream_t s) {
  const long n = (long)npos * (hd / 2);
  k_rope_table<<<(unsigned)((n + 255) / 256), 256, 0, s>>>(cs, npos, hd, (double)base);
  return hipGetLastError();
}

// --------------------------------------------------------------- row tables
__global__ void k_row_tables(Branches br, int P, const int32_t *cand_ids, int vocab,
                             int32_t *flags, int32_t *row_lo, int32_t *row_pos,
                             int32_t *lm_tgt) {
  const int t = blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= br.cu[br.M]) return;
  int m = 0;
  while (br.cu[m + 1] <= t) ++m;
  const int j = t - br.cu[m];
  int id = cand_ids[(long)m * br.cmax + j];
  if (id < 0 || id >= vocab) {
    atomicOr(flags, kFlagBadId);
    id = 0;
  }
  row_lo[t] = br.cu[m];
  row_pos[t] = P + j;
  lm_tgt[t] = id;
}

hipError_t launch_row_tables(const Branches &br, int P, const int32_t *cand_ids, int vocab,
                             int32_t *flags, int32_t *row_lo, int32_t *row_pos,
                             int32_t *lm_tgt, hipStream_t s) {
  const int T = br.cu[br.M];
  if (T == 0) return hipSuccess;
  k_row_tables<<<(T + 255) / 256, 256, 0, s>>>(br, P, cand_ids, vocab, flags, row_lo, row_pos,
                                               lm_tgt);
  return hipGetLastError();
}

// Row tables of a draft call. Prompt row t of branch m at offset j sits at
// decode-cache position m S + j (a fixed stride S per branch, room for the
// prompt and the new tokens): row_lo = m S, row_pos = P + j (rotary),
// cache_row = m S + j, lm_tgt = the prompt id (clamped).
__global__ void k_draft_rows(Branches br, int P, int S, const int32_t *ids, int vocab,
                             int32_t *flags, int32_t *row_lo, int32_t *row_pos,
                             int32_t *cache_row, int32_t *lm_tgt) {
  const int t = blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= br.cu[br.M]) return;
  int m = 0;
  while (br.cu[m + 1] <= t) ++m;
  const int j = t - br.cu[m];
  int id = ids[(long)m * br.cmax + j];
  if (id < 0 || id >= vocab) {
    atomicOr(flags, kFlagBadId);
    id = 0;
  }
  row_lo[t] = m * S;
  row_pos[t] = P + j;
  cache_row[t] = m * S + j;
  lm_tgt[t] = id;
}

hipError_t launch_draft_rows(const Branches &br, int P, int S, const int32_t *ids, int vocab,
                             int32_t *flags, int32_t *row_lo, int32_t *row_pos,
                             int32_t *cache_row, int32_t *lm_tgt, hipStream_t s) {
  const int T = br.cu[br.M];
  k_draft_rows<<<(T + 255) / 256, 256, 0, s>>>(br, P, S, ids, vocab, flags, row_lo, row_pos,
                                               cache_row, lm_tgt);
  return hipGetLastError();
}

// Decode step s >= 1: row m is new token s - 1 of branch m, at branch offset
// n_m + s - 1.
__global__ void k_draft_step(Branches br, int P, int S, int step, int32_t *row_lo,
                             int32_t *row_pos, int32_t *cache_row) {
  const int m = blockIdx.x * blockDim.x + threadIdx.x;
  if (m >= br.M) return;
  const int j = br.cu[m + 1] - br.cu[m] + step - 1;
  row_lo[m] = m * S;
  row_pos[m] = P + j;
  cache_row[m] = m * S + j;
}

hipError_t launch_draft_step(const Branches &br, int P, int S, int step, int32_t *row_lo,
                             int32_t *row_pos, int32_t *cache_row, hipStream_t s) {
  k_draft_step<<<(br.M + 63) / 64, 64, 0, s>>>(br, P, S, step, row_lo, row_pos, cache_row);
  return hipGetLastError();
}

// Greedy pick per row from the LM-head partials (chunks in vocabulary order,
// each holding its lowest best index): tokens[m][step] and the next inputs.
// Block per row: threads stride over the chunks, then waves and blocks keep
// the largest value and, among equal values, the lowest index.
__device__ __forceinline__ void keep_best(float &v, int &i, float v2, int i2) {
  if (i2 >= 0 && (i < 0 || v2 > v || (v2 == v && i2 < i))) {
    v = v2;
    i = i2;
  }
}

__global__ __launch_bounds__(1024) void k_argmax_merge(const float2 *part, int nchunks, int M,
                                                       int n_new, int step, int32_t *tokens,
                                                       int32_t *next_ids) {
  __shared__ float sv[16];
  __shared__ int si[16];
  const int m = blockIdx.x, lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  float best = -INFINITY;
  int bi = -1;
  for (int c = threadIdx.x; c < nchunks; c += 1024) {
    const float2 p = part[(long)c * M + m];
    keep_best(best, bi, p.x, __float_as_int(p.y));
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1)
    keep_best(best, bi, __shfl_xor(best, o, 64), __shfl_xor(bi, o, 64));
  if (lane == 0) {
    sv[w] = best;
    si[w] = bi;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int i = 1; i < 16; ++i) keep_best(best, bi, sv[i], si[i]);
    tokens[(long)m * n_new + step] = bi;
    next_ids[m] = bi;
  }
}

hipError_t launch_argmax_merge(const float2 *part, int nchunks, int M, int n_new, int step,
                               int32_t *tokens, int32_t *next_ids, hipStream_t s) {
  k_argmax_merge<<<M, 1024, 0, s>>>(part, nchunks, M, n_new, step, tokens, next_ids);
  return hipGetLastError();
}

// ---------------------------------------------------------- call validator
// The status word of a checked call: cleared at its start, bits set by the
// kernels that meet a bad id or a non-finite result, read once at its end.
__global__ void k_flags_clear(int32_t *flags) {
  if (threadIdx.x == 0) flags[0] = 0;
}

hipError_t launch_flags_clear(int32_t *flags, hipStream_t s) {
  k_flags_clear<<<1, 64, 0, s>>>(flags);
  return hipGetLastError();
}

// Sets kFlagNonFinite if any of x[0 .. n) is NaN or infinite.
__global__ __launch_bounds__(256) void k_check_finite(const float *x, long n, int32_t *flags) {
  bool bad = false;
  for (long i = (long)blockIdx.x * 256 + threadIdx.x; i < n; i += (long)gridDim.x * 256)
    bad |= !isfinite(x[i]);
  if (__any(bad) && (threadIdx.x & 63) == 0) atomicOr(flags, kFlagNonFinite);
}

hipError_t launch_check_finite(const float *x, long n, int32_t *flags, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  const long blocks = std::min<long>((n + 255) / 256, 1024);
  k_check_finite<<<(unsigned)blocks, 256, 0, s>>>(x, n, flags);
  return hipGetLastError();
}

// ---------------------------------------------------------------- embedding
template <typename T>
__global__ void k_embed_prefix(const T *visual, int n_visual, const int32_t *ids,
                               const T *embed, int vocab, int d, float *x, int32_t *flags) {
  const int p = blockIdx.x;
  const T *src;
  if (p < n_visual) {
    src = visual + (long)p * d;
  } else {
    int id = ids[p - n_visual];
    if (id < 0 || id >= vocab) {
      if (threadIdx.x == 0) atomicOr(flags, kFlagBadId);
      id = 0;
    }
    src = embed + (long)id * d;
  }
  float *dst = x + (long)p * d;
  for (int c = threadIdx.x; c < d; c += blockDim.x) dst[c] = to_f32(src[c]);
}

template <typename T>
hipError_t launch_embed_prefix(const T *visual, int n_visual, const int32_t *ids, int n_text,
                               const T *embed, int vocab, int d, float *x, int32_t *flags,
                               hipStream_t s) {
  const int P = n_visual + n_text;
  k_embed_prefix<T><<<P, 256, 0, s>>>(visual, n_visual, ids, embed, vocab, d, x, flags);
  return hipGetLastError();
}

template <typename T>
__global__ void k_embed_rows(const int32_t *ids, const T *embed, int d, float *x) {
  const int t = blockIdx.x;
  const T *src = embed + (long)ids[t] * d;
  float *dst = x + (long)t * d;
  for (int c = threadIdx.x; c < d; c += blockDim.x) dst[c] = to_f32(src[c]);
}

// Candidate rows use the row table's clamped ids (lm_tgt holds cand_ids[m][j]).
template <typename T>
hipError_t launch_embed_rows(const int32_t *ids, int rows, const T *embed, int d, float *x,
                             hipStream_t s) {
  if (rows == 0) return hipSuccess;
  k_embed_rows<T><<<rows, 256, 0, s>>>(ids, embed, d, x);
  return hipGetLastError();
}

// ------------------------------------------------------------------ RMSNorm
// One row by a 256-thread block: y = x / sqrt(mean(x^2) + eps) * g (+ the
// remainder half when split == 2). Rows of d % 4 == 0, d <= 8192 are read once
// as float4 and kept in registers; others take the scalar two-pass path.
template <typename TW, typename TA>
__device__ __forceinline__ void norm_row(const float *src, const TW *g, int d, float eps,
                                         TA *dst, float *red, int split = 1) {
  constexpr int NV = 8;  // float4 per thread: d <= 256 * 4 * NV
  if (d % 4 == 0 && d <= 256 * 4 * NV) {
    const int n4 = d / 4;
    float4 v[NV];
    float ss = 0.f;
#pragma unroll
    for (int i = 0; i < NV; ++i) {
      const int c4 = threadIdx.x + 256 * i;
      v[i] = c4 < n4 ? reinterpret_cast<const float4 *>(src)[c4] : make_float4(0.f, 0.f, 0.f, 0.f);
      ss += v[i].x * v[i].x + v[i].y * v[i].y + v[i].z * v[i].z + v[i].w * v[i].w;
    }
    ss = block_sum256(ss, red);
    const float r = rsqrtf(ss / (float)d + eps);
#pragma unroll
    for (int i = 0; i < NV; ++i) {
      const int c4 = threadIdx.x + 256 * i;
      if (c4 >= n4) break;
      const float x[4] = {v[i].x, v[i].y, v[i].z, v[i].w};
      TA hi[4], lo[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const float y = x[e] * r * to_f32(g[4 * c4 + e]);
        hi[e] = from_f32<TA>(y);
        lo[e] = from_f32<TA>(y - to_f32(hi[e]));
      }
      // Four outputs per store.
      struct alignas(4 * sizeof(TA)) Q4 { TA v[4]; };
      *reinterpret_cast<Q4 *>(dst + 4 * c4) = Q4{{hi[0], hi[1], hi[2], hi[3]}};
      if (split == 2) *reinterpret_cast<Q4 *>(dst + d + 4 * c4) = Q4{{lo[0], lo[1], lo[2], lo[3]}};
    }
    return;
  }
  float ss = 0.f;
  for (int c = threadIdx.x; c < d; c += 256) {
    const float v = src[c];
    ss += v * v;
  }
  ss = block_sum256(ss, red);
  const float r = rsqrtf(ss / (float)d + eps);
  for (int c = threadIdx.x; c < d; c += 256) {
    const float v = src[c] * r * to_f32(g[c]);
    const TA hi = from_f32<TA>(v);
    dst[c] = hi;
    if (split == 2) dst[d + c] = from_f32<TA>(v - to_f32(hi));
  }
}

template <typename TW, typename TA>
__global__ __launch_bounds__(256) void k_rmsnorm(const float *x, const TW *g, int d, float eps,
                                                 TA *y, int split) {
  __shared__ float red[4];
  const long r = blockIdx.x;
  norm_row(x + r * d, g, d, eps, y + r * d * split, red, split);
}

template <typename TW, typename TA>
hipError_t launch_rmsnorm(const float *x, const TW *g, int rows, int d, float eps, TA *y,
                          int split, hipStream_t s) {
  if (rows == 0) return hipSuccess;
  k_rmsnorm<TW, TA><<<rows, 256, 0, s>>>(x, g, d, eps, y, split);
  return hipGetLastError();
}

template <typename TW, typename TA>
__global__ __launch_bounds__(256) void k_lm_inputs(const float *x, const float *h_last,
                                                   const int32_t *row_lo, const TW *g, int d,
                                                   float eps, TA *y) {
  __shared__ float red[4];
  const int t = blockIdx.x;
  const float *src = (row_lo[t] == t) ? h_last : x + (long)(t - 1) * d;
  norm_row(src, g, d, eps, y + (long)t * d, red);
}

template <typename TW, typename TA>
hipError_t launch_lm_inputs(const float *x, const float *h_last, const int32_t *row_lo,
                            const TW *g, int T_rows, int d, float eps, TA *y, hipStream_t s) {
  if (T_rows == 0) return hipSuccess;
  k_lm_inputs<TW, TA><<<T_rows, 256, 0, s>>>(x, h_last, row_lo, g, d, eps, y);
  return hipGetLastError();
}

// Draft prompt stage: block m normalises the last prompt row of branch m.
template <typename TW, typename TA>
__global__ __launch_bounds__(256) void k_branch_last_norm(const float *x, Branches br,
                                                          const TW *g, int d, float eps,
                                                          TA *y) {
  __shared__ float red[4];
  const int m = blockIdx.x;
  norm_row(x + (long)(br.cu[m + 1] - 1) * d, g, d, eps, y + (long)m * d, red);
}

template <typename TW, typename TA>
hipError_t launch_branch_last_norm(const float *x, const Branches &br, const TW *g, int d,
                                   float eps, TA *y, hipStream_t s) {
  k_branch_last_norm<TW, TA><<<br.M, 256, 0, s>>>(x, br, g, d, eps, y);
  return hipGetLastError();
}

// Reliability rows: block b normalises the last row of branch b % M.
template <typename TW, typename TA>
__global__ __launch_bounds__(256) void k_last_inputs(const float *x, Branches br, const TW *g,
                                                     int d, float eps, int yes_id, int no_id,
                                                     TA *y, int32_t *lm_tgt) {
  __shared__ float red[4];
  const int b = blockIdx.x, m = b % br.M;
  const int t = br.cu[m + 1] - 1;  // every branch has at least one row
  norm_row(x + (long)t * d, g, d, eps, y + (long)b * d, red);
  if (threadIdx.x == 0) lm_tgt[b] = b < br.M ? yes_id : no_id;
}

template <typename TW, typename TA>
hipError_t launch_last_inputs(const float *x, const Branches &br, const TW *g, int d, float eps,
                              int yes_id, int no_id, TA *y, int32_t *lm_tgt, hipStream_t s) {
  k_last_inputs<TW, TA><<<2 * br.M, 256, 0, s>>>(x, br, g, d, eps, yes_id, no_id, y, lm_tgt);
  return hipGetLastError();
}

// ----------------------------------------------------- LSE merge and gather
// Log-sum-exp of up to 16 LM-head rows (of T) over their vocabulary chunks, by
// a block of NT threads: thread i takes row i % 16 (`t`, -1: none) and every
// NT / 16th chunk, so a load covers the adjacent rows' partials of 4 chunks (a
// wave per row read 64 lines per load and one 8-byte value of each); eight
// loads in flight, rescaled to the thread's running maximum, then a tree over
// the NT / 16 threads of a row. Returns the row's value to thread i < 16.
template <int NT>
__device__ __forceinline__ float block_lse(const float2 *part, int nchunks, int T, int t,
                                           float2 *red) {
  constexpr int U = 8, G = NT / 16;
  const int tid = threadIdx.x;
  float mx = -INFINITY, sum = 0.f;
  if (t >= 0) {
    for (int c0 = tid >> 4; c0 < nchunks; c0 += G * U) {
      float2 p[U];
#pragma unroll
      for (int u = 0; u < U; ++u)
        p[u] = c0 + G * u < nchunks ? part[(long)(c0 + G * u) * T + t]
                                    : make_float2(-INFINITY, 0.f);
      float m = mx;
#pragma unroll
      for (int u = 0; u < U; ++u) m = fmaxf(m, p[u].x);
      if (mx != m) sum = sum == 0.f ? 0.f : sum * __expf(mx - m);
      mx = m;
#pragma unroll
      for (int u = 0; u < U; ++u) sum += p[u].y == 0.f ? 0.f : p[u].y * __expf(p[u].x - m);
    }
  }
  __syncthreads();  // an earlier call's values are used
  red[tid] = make_float2(mx, sum);
  __syncthreads();
#pragma unroll
  for (int o = NT / 2; o >= 16; o >>= 1) {
    if (tid < o) {
      const float2 x = red[tid], y = red[tid + o];
      const float m = fmaxf(x.x, y.x);
      red[tid] = make_float2(m, (x.y == 0.f ? 0.f : x.y * __expf(x.x - m)) +
                                    (y.y == 0.f ? 0.f : y.y * __expf(y.x - m)));
    }
    __syncthreads();
  }
  return tid < 16 ? red[tid].x + __logf(red[tid].y) : 0.f;
}

// One block: the 2M rows (a branch's Yes row m, its No row M + m) 16 at a
// time; then thread 0 takes the maximum reliability and every thread marks its
// branches (Eq. 13).
constexpr int RF_T = 1024;
__global__ __launch_bounds__(RF_T) void k_reliability_finish(int M, const float2 *part,
                                                            int nchunks, const float *tgt,
                                                            float delta, float *lp_yes_no,
                                                            float *rel, int32_t *keep) {
  __shared__ float lp[2 * kMaxCands], r[kMaxCands];
  __shared__ float best;
  __shared__ float2 red[RF_T];
  for (int i0 = 0; i0 < 2 * M; i0 += 16) {
    const int i = i0 + (threadIdx.x & 15);
    const float lse = block_lse<RF_T>(part, nchunks, 2 * M, i < 2 * M ? i : -1, red);
    if (threadIdx.x < 16 && i < 2 * M) lp[i] = tgt[i] - lse;
  }
  __syncthreads();
  for (int m = threadIdx.x; m < M; m += RF_T) {
    const float ly = lp[m], ln = lp[M + m], v = 1.f / (1.f + expf(ln - ly));
    lp_yes_no[2 * m] = ly;
    lp_yes_no[2 * m + 1] = ln;
    rel[m] = v;
    r[m] = v;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    float b = r[0];
    for (int m = 1; m < M; ++m) b = fmaxf(b, r[m]);
    best = b;
  }
  __syncthreads();
  for (int m = threadIdx.x; m < M; m += RF_T) keep[m] = r[m] >= best - delta ? 1 : 0;
}

hipError_t launch_reliability_finish(int M, const float2 *part, int nchunks,
                                     const float *tgt_logit, float delta, float *lp_yes_no,
                                     float *rel, int32_t *keep, hipStream_t s) {
  k_reliability_finish<<<1, RF_T, 0, s>>>(M, part, nchunks, tgt_logit, delta, lp_yes_no, rel,
                                         keep);
  return hipGetLastError();
}

// --------------------------------------------- entity alignment and choice
// cos = (e . f) / (|e| |f|), 0 if either norm is 0.
typedef float f32x4u __attribute__((ext_vector_type(4), aligned(4)));

// Few frames: block m (16 waves) takes draft m against every frame, a wave
// four frames at a time, the lanes four coordinates each. Latency-bound: the
// loads of the four frames are in flight together and the sums stay in
// registers (one frame after the other, with LDS permutes for the sums, took
// 11 us for 8 x 64 x 768; now 5.2 us).
__global__ __launch_bounds__(1024) void k_align(const float *ent, const float *frames, int NF,
                                                int D, float *align) {
  __shared__ float red[16];
  const int m = blockIdx.x, w = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const float *e = ent + (long)m * D;
  auto ld = [&](const float *p, int c) {
    f32x4 v = {0.f, 0.f, 0.f, 0.f};
    if (c + 3 < D)
      v = *reinterpret_cast<const f32x4u *>(p + c);
    else
#pragma unroll
      for (int j = 0; j < 4; ++j)
        if (c + j < D) v[j] = p[c + j];
    return v;
  };
  float best = -INFINITY;
  for (int f = w; f < NF; f += 64) {
    float ee = 0.f, ef[4] = {0.f, 0.f, 0.f, 0.f}, ff[4] = {0.f, 0.f, 0.f, 0.f};
    const float *fr[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) fr[j] = frames + (long)min(f + 16 * j, NF - 1) * D;
    for (int c0 = 4 * lane; c0 < D; c0 += 768) {
      f32x4 x[3], y[3][4];
#pragma unroll
      for (int i = 0; i < 3; ++i) {
        x[i] = ld(e, c0 + 256 * i);
#pragma unroll
        for (int j = 0; j < 4; ++j) y[i][j] = ld(fr[j], c0 + 256 * i);
      }
#pragma unroll
      for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          ee += x[i][k] * x[i][k];
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            ef[j] += x[i][k] * y[i][j][k];
            ff[j] += y[i][j][k] * y[i][j][k];
          }
        }
    }
    ee = wave_sum(ee);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const float den = sqrtf(ee) * sqrtf(wave_sum(ff[j]));
      const float dot = wave_sum(ef[j]);
      best = fmaxf(best, den > 0.f ? dot / den : 0.f);  // (a repeated last frame: no change)
    }
  }
  if (lane == 0) red[w] = best;
  __syncthreads();
  if (threadIdx.x == 0) {
    float b = red[0];
#pragma unroll
    for (int i = 1; i < 16; ++i) b = fmaxf(b, red[i]);
    align[m] = b;
  }
}

// Many frames: a block of 16 waves takes 16 drafts x 64 frames at a time as
// fp32 matrix products: wave w has frames 16 (w % 4) .. + 15 of the 64 and
// every fourth 16-wide piece of D; the partial products and the rows' squares
// meet in LDS. 64 drafts x 2048 frames x 1024: 645 us with a block per draft and
// a frame at a time, now 23 us.
constexpr int AL_M = 16, AL_F = 64, AL_T = 1024;

struct AlignTile {
  float red[16][256];
  float ee[4][16], ff[4][4][16];
};

// The largest cosine of drafts m0 .. m0 + 15 over frames f0, f0 + AL_F, ...
// (step frames apart, below NF): thread t < 64 gets draft m0 + t / 4's maximum
// over the 16-frame groups t % 4 of its tiles.
__device__ __forceinline__ float align_tiles(AlignTile &s, const float *ent, const float *frames,
                                             int M, long NF, int D, int m0, long f0, long step) {
  __shared__ float best[AL_M][4];
  const int t = threadIdx.x, w = t >> 6, lane = t & 63, c16 = lane & 15, sub = 4 * (lane >> 4);
  const int fg = w & 3, kq = w >> 2, np = (D + 15) / 16, nfull = D / 16;
  const float *ep = ent + (long)min(m0 + c16, M - 1) * D + sub;
  if (t < AL_M * 4) best[t >> 2][t & 3] = -INFINITY;
  constexpr int U = 4;  // pieces in flight
  for (long f = f0; f < NF; f += step) {
    const float *fp = frames + min(f + 16 * fg + c16, NF - 1) * D + sub;
    // The matrix products add four terms each; what follows is a tree per piece.
    // One chain over the wave's share of D lost twice the bits of the other form's
    // short lane sums (1.4e-7 against 7.5e-8 for 768 dimensions; now 7.8e-8).
    const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
    f32x4 acc = zero;
    float ee = 0.f, ff = 0.f;
    auto add = [&](f32x4 e, f32x4 x) {
      ee += e[0] * e[0] + e[1] * e[1] + e[2] * e[2] + e[3] * e[3];
      ff += x[0] * x[0] + x[1] * x[1] + x[2] * x[2] + x[3] * x[3];
      f32x4 s[4];
#pragma unroll
      for (int j = 0; j < 4; ++j)
        s[j] = __builtin_amdgcn_mfma_f32_16x16x4f32(e[j], x[j], zero, 0, 0, 0);
      acc += (s[0] + s[1]) + (s[2] + s[3]);
    };
    for (int p = kq; p < nfull; p += 4 * U) {
      f32x4 e[U], x[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int k = 16 * min(p + 4 * u, nfull - 1);
        e[u] = *reinterpret_cast<const f32x4u *>(ep + k);
        x[u] = *reinterpret_cast<const f32x4u *>(fp + k);
      }
#pragma unroll
      for (int u = 0; u < U; ++u)
        if (p + 4 * u < nfull) add(e[u], x[u]);
    }
    if (np > nfull && nfull % 4 == kq) {  // the last, partial piece
      f32x4 e, x;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const bool in = 16 * nfull + sub + j < D;
        e[j] = in ? ep[16 * nfull + j] : 0.f;
        x[j] = in ? fp[16 * nfull + j] : 0.f;
      }
      add(e, x);
    }
    ee += __shfl_xor(ee, 16, 64);
    ee += __shfl_xor(ee, 32, 64);
    ff += __shfl_xor(ff, 16, 64);
    ff += __shfl_xor(ff, 32, 64);
    __syncthreads();  // the previous tile's values are used
#pragma unroll
    for (int r = 0; r < 4; ++r) s.red[w][64 * r + lane] = acc[r];
    if (lane < 16) {
      s.ff[fg][kq][lane] = ff;
      if (fg == 0) s.ee[kq][lane] = ee;
    }
    __syncthreads();
    // Thread t: 16-frame group t / 256, draft row 4 ((t % 64) / 16) +
    // (t % 256) / 64, frame column t % 16.
    const int g = t >> 8, el = t & 255, row = 4 * ((el & 63) >> 4) + (el >> 6);
    const float dot = (s.red[g][el] + s.red[g + 4][el]) + (s.red[g + 8][el] + s.red[g + 12][el]);
    const float se = (s.ee[0][row] + s.ee[1][row]) + (s.ee[2][row] + s.ee[3][row]);
    const float sf = (s.ff[g][0][c16] + s.ff[g][1][c16]) + (s.ff[g][2][c16] + s.ff[g][3][c16]);
    const float den = sqrtf(se) * sqrtf(sf);
    float v = f + 16 * g + c16 < NF ? (den > 0.f ? dot / den : 0.f) : -INFINITY;
#pragma unroll
    for (int o = 1; o < 16; o <<= 1) v = fmaxf(v, __shfl_xor(v, o, 64));
    if (c16 == 0) best[row][g] = fmaxf(best[row][g], v);
  }
  __syncthreads();
  return t < AL_M * 4 ? best[t >> 2][t & 3] : -INFINITY;
}

// The final choice by wave 0 from the alignments in LDS. An argmax takes the
// first allowed index if its value is NaN (nothing compares greater), else
// the lowest index of the largest value.
__device__ __forceinline__ void choose(const float *rel, const float *al, int M, float delta,
                                       int strategy, int32_t *choice) {
  constexpr int E = kMaxCands / 64;
  if (threadIdx.x >= 64) return;
  const int lane = threadIdx.x;
  float filt[E], rank[E];
  float mx = -INFINITY;
#pragma unroll
  for (int e = 0; e < E; ++e) {
    const int m = lane + 64 * e;
    const float r = m < M ? rel[m] : -INFINITY, a = m < M ? al[m] : -INFINITY;
    filt[e] = strategy == 0 ? r : a;
    rank[e] = strategy == 1 ? r + a : strategy == 0 ? a : r;
    mx = fmaxf(mx, filt[e]);
  }
  mx = wave_max(mx);
  int first = 0x7fffffff, bi = 0x7fffffff;
  float first_v = 0.f, bv = -INFINITY;
#pragma unroll
  for (int e = 0; e < E; ++e) {
    const int m = lane + 64 * e;
    const bool ok = m < M && (strategy == 1 || filt[e] >= mx - delta);
    if (ok && m < first) {
      first = m;
      first_v = rank[e];
    }
    if (ok && !isnan(rank[e]) && (bi == 0x7fffffff || rank[e] > bv)) {
      bv = rank[e];
      bi = m;
    }
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    const int f2 = __shfl_xor(first, o, 64), i2 = __shfl_xor(bi, o, 64);
    const float fv2 = __shfl_xor(first_v, o, 64), v2 = __shfl_xor(bv, o, 64);
    if (f2 < first) {
      first = f2;
      first_v = fv2;
    }
    if (i2 != 0x7fffffff && (bi == 0x7fffffff || v2 > bv || (v2 == bv && i2 < bi))) {
      bv = v2;
      bi = i2;
    }
  }
  if (lane == 0) *choice = first == 0x7fffffff ? -1 : isnan(first_v) ? first : bi;
}

__global__ __launch_bounds__(64) void k_choose(const float *rel, const float *align, int M,
                                               float delta, int strategy, int32_t *choice) {
  choose(rel, align, M, delta, strategy, choice);
}

// Blocks over (frame tiles, draft tiles) take maxima
// into align as order-preserving integers (atomics), counting themselves in
// *choice; the last one decodes them and chooses. k_align_init sets both.
__device__ __forceinline__ int32_t ordered_bits(float v) {
  const int32_t i = __float_as_int(v);
  return i >= 0 ? i : i ^ 0x7fffffff;
}

__global__ void k_align_init(int M, int32_t *align, int32_t *choice) {
  for (int m = threadIdx.x; m < M; m += blockDim.x) align[m] = ordered_bits(-INFINITY);
  if (threadIdx.x == 0) *choice = 0;
}

__global__ __launch_bounds__(AL_T) void k_align_many(const float *ent, const float *frames, int M,
                                                     int NF, int D, const float *rel, float delta,
                                                     int strategy, float *align,
                                                     int32_t *choice) {
  __shared__ AlignTile s;
  __shared__ float al[kMaxCands];
  __shared__ int32_t finished;
  const int t = threadIdx.x, m0 = blockIdx.y * AL_M;
  float v = align_tiles(s, ent, frames, M, NF, D, m0, (long)blockIdx.x * AL_F,
                        (long)gridDim.x * AL_F);
  v = fmaxf(v, __shfl_xor(v, 1, 64));
  v = fmaxf(v, __shfl_xor(v, 2, 64));
  int32_t *bits = reinterpret_cast<int32_t *>(align);
  if (t < AL_M * 4) {  // wave 0
    if ((t & 3) == 0 && m0 + (t >> 2) < M)
      __hip_atomic_fetch_max(&bits[m0 + (t >> 2)], ordered_bits(v), __ATOMIC_RELAXED,
                             __HIP_MEMORY_SCOPE_AGENT);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // the maxima are in
    if (t == 0)
      finished = __hip_atomic_fetch_add(choice, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  __syncthreads();
  if (finished != (int)(gridDim.x * gridDim.y) - 1) return;  // uniform per block
  if (t < M) {
    const int32_t i =
        __hip_atomic_load(&bits[t], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    const float x = __int_as_float(i >= 0 ? i : i ^ 0x7fffffff);
    al[t] = x;
    align[t] = x;
  }
  __syncthreads();
  choose(rel, al, M, delta, strategy, choice);
}

hipError_t launch_align_select(const float *ent, const float *frames, int M, int NF, int D,
                               const float *rel, float delta, int strategy, float *align,
                               int32_t *choice, hipStream_t s) {
  // A block per draft walks the frames at 3 to 4.5 us per 64 of them; the tiled
  // form takes 11 to 21 us up to 2048 frames. They cross near 192 frames: 128
  // frames of 768 10 against 17 us, 170 of 1024 18 against 19, 256 of 512 16
  // against 13.
  if (NF <= 192) {
    k_align<<<M, 1024, 0, s>>>(ent, frames, NF, D, align);
    k_choose<<<1, 64, 0, s>>>(rel, align, M, delta, strategy, choice);
  } else {
    k_align_init<<<1, 256, 0, s>>>(M, reinterpret_cast<int32_t *>(align), choice);
    const dim3 grid((unsigned)std::min<long>(((long)NF + AL_F - 1) / AL_F, 2048),
                    (M + AL_M - 1) / AL_M);
    k_align_many<<<grid, AL_T, 0, s>>>(ent, frames, M, NF, D, rel, delta, strategy, align, choice);
  }
  return hipGetLastError();
}

// Block per 16 output slots (m, j).
__global__ __launch_bounds__(256) void k_lse_gather(Branches br, const float2 *part,
                                                    int nchunks, const float *tgt_logit,
                                                    float *logprobs) {
  __shared__ float2 red[256];
  const int slot = blockIdx.x * 16 + (threadIdx.x & 15);
  const bool in = slot < br.M * br.cmax;
  int t = -1;
  if (in) {
    const int m = slot / br.cmax, j = slot % br.cmax;
    if (j < br.cu[m + 1] - br.cu[m]) t = br.cu[m] + j;
  }
  const float lse = block_lse<256>(part, nchunks, br.cu[br.M], t, red);
  if (threadIdx.x < 16 && in) logprobs[slot] = t < 0 ? 0.f : tgt_logit[t] - lse;
}

hipError_t launch_lse_gather(const Branches &br, const float2 *part, int nchunks,
                             const float *tgt_logit, float *logprobs, hipStream_t s) {
  const int slots = br.M * br.cmax;
  k_lse_gather<<<(slots + 15) / 16, 256, 0, s>>>(br, part, nchunks, tgt_logit, logprobs);
  return hipGetLastError();
}

// ------------------------------------------------- per-candidate sum, argmax
// One block; wave w sums candidates w, w+4, ... with a fixed lane order, then
// thread 0 takes the first index of the largest score (Eq. 7).
__global__ __launch_bounds__(256) void k_reduce_select(Branches br, const float *logprobs,
                                                       float *scores, int32_t *argmax) {
  __shared__ float sc[kMaxCands];
  const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
  for (int m = w; m < br.M; m += 4) {
    const int n = br.cu[m + 1] - br.cu[m];
    float v = 0.f;
    for (int j = lane; j < n; j += 64) v += logprobs[(long)m * br.cmax + j];
    v = wave_sum(v);
    if (lane == 0) {
      sc[m] = v;
      scores[m] = v;
    }
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    int best = 0;
    for (int m = 1; m < br.M; ++m)
      if (sc[m] > sc[best]) best = m;
    *argmax = best;
  }
}

hipError_t launch_reduce_select(const Branches &br, const float *logprobs, float *scores,
                                int32_t *argmax, hipStream_t s) {
  k_reduce_select<<<1, 256, 0, s>>>(br, logprobs, scores, argmax);
  return hipGetLastError();
}

#define VSR_INST(T)                                                                          \
  template hipError_t launch_embed_prefix<T>(const T *, int, const int32_t *, int, const T *, \
                                             int, int, float *, int32_t *, hipStream_t);    \
  template hipError_t launch_embed_rows<T>(const int32_t *, int, const T *, int, float *,     \
                                           hipStream_t);
VSR_INST(float)
VSR_INST(bf16)
#undef VSR_INST
#define VSR_INST2(TW, TA)                                                                     \
  template hipError_t launch_rmsnorm<TW, TA>(const float *, const TW *, int, int, float,      \
                                             TA *, int, hipStream_t);                         \
  template hipError_t launch_lm_inputs<TW, TA>(const float *, const float *, const int32_t *, \
                                               const TW *, int, int, float, TA *, hipStream_t); \
  template hipError_t launch_last_inputs<TW, TA>(const float *, const Branches &, const TW *, \
                                                 int, float, int, int, TA *, int32_t *,       \
                                                 hipStream_t);                                \
  template hipError_t launch_branch_last_norm<TW, TA>(const float *, const Branches &,        \
                                                      const TW *, int, float, TA *,           \
                                                      hipStream_t);
VSR_INST2(float, float)
VSR_INST2(bf16, f16)
#undef VSR_INST2

}  // namespace vsr
