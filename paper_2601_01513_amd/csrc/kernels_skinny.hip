// Projections of a few rows (decode steps of the drafter, the prefix pass's
// last-row layer): Y = A W^T with A [rows <= 32][K] fp16 activations and W
// [N][K] weights. With so few rows the product is a stream over the weights,
// bound by HBM bandwidth, not by the matrix cores: the kernel's job is to keep
// enough weight bytes in flight on every CU, in as few launches as possible.
//
// Layout of the work: a wave owns 16 weight rows and one K slice; it streams
// its rows in 256-wide K steps (eight 16-byte weight loads per lane and the
// matching activation loads, all issued before the first use), each 32-wide
// piece feeding one v_mfma_f32_16x16x32_f16 with the weights as the 16-row
// operand and up to 16 activation rows as the 16-column operand (a second
// product per row group for the fp16 remainder half of precise-layer rows, a
// second row group for 17..32 rows). A block is four waves over one group of
// 64 weight rows and the same K slice, so their activation loads hit the same
// cache lines.
//
// Up to 8 rows of the usual widths take k_few below, one launch per projection;
// what follows is the form of up to 32 rows and any width.
//
// The K slices write fp32 partials part[s][row][n]; a small reduce kernel
// sums them in slice order (deterministic) and applies the epilogue: residual
// add (+ the RMSNorm that follows), SwiGLU, or rotary + cache scatter. (A
// reduction by the last-arriving block of each group would save that launch,
// but its cross-block release is an L2 writeback per block on this chip,
// which costs more than the launch.)
#include <algorithm>

#include "common.h"

namespace vsr {

namespace {

constexpr int SK_ROWS = 64;   // weight rows per block (16 per wave)
constexpr int SK_STEP = 256;  // K per unrolled step
constexpr int SK_U = SK_STEP / 32;

__device__ __forceinline__ f16x8 as_h8(u32x4 v) { return __builtin_bit_cast(f16x8, v); }

// Eight bf16 weights -> fp16 with the tile GEMMs' rounding (exact for
// magnitudes in [2^-17, 65504]).
__device__ __forceinline__ u32x4 sk_bf16_to_f16(u32x4 v) {
  u32x4 r;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const float lo = __uint_as_float(v[i] << 16);
    const float hi = __uint_as_float(v[i] & 0xFFFF0000u);
    r[i] = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_pkrtz(lo, hi));
  }
  return r;
}

__device__ __forceinline__ u32x4 ld16(const void *p) {
  return *reinterpret_cast<const u32x4 *>(p);
}

// Sum of the ksplit slices of element i in slice order. All loads are issued
// before the first add (slices past ksplit re-load the last one and add 0).
__device__ __forceinline__ float sum_slices(const float *part, int ksplit, long stride,
                                            long i) {
  float v[kSkinnyMaxSplit];
#pragma unroll
  for (int s = 0; s < kSkinnyMaxSplit; ++s) v[s] = part[min(s, ksplit - 1) * stride + i];
  float acc = v[0];
#pragma unroll
  for (int s = 1; s < kSkinnyMaxSplit; ++s) acc += s < ksplit ? v[s] : 0.f;
  return acc;
}

// RG row groups of 16 activation rows; AS = 2: rows are [hi | lo] of width 2K.
// NW groups of 16 weight rows per wave: two halve the activation loads per
// weight byte but cost occupancy. SK_LSE takes two (16 rows of the 7B head in
// bf16: 267 us against 288), the greedy head of a few drafts one (3 rows of
// the 3B drafter's: 114 us against 125).
// SK_ARGMAX and SK_LSE (LM head, one K slice): instead of the products, each
// block writes, per row, over its 64 NW outputs, part[blockIdx.x][row] = (largest
// value, its lowest index as bits) or (largest value m, sum of exp(l - m));
// SK_LSE also writes the row's target logit if it is among them.
enum { SK_PART, SK_ARGMAX, SK_LSE };
template <int RG, int AS, bool WCVT, int OUT, int NW = 1>
__global__ __launch_bounds__(256) void k_skinny(const f16 *__restrict__ A, int rows,
                                                const uint16_t *__restrict__ W, int N, int K,
                                                int ksplit, float *__restrict__ part,
                                                const int32_t *__restrict__ tgt,
                                                float *__restrict__ tgt_logit) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int b = blockIdx.x, s = blockIdx.y;
  const int n0 = SK_ROWS * NW * b + 16 * NW * w;
  // Slices are whole 256-wide steps (only the last one may end short).
  const int nsteps = (K + SK_STEP - 1) / SK_STEP;
  const int k0 = (int)((long)nsteps * s / ksplit) * SK_STEP;
  const int k1 = min(K, (int)((long)nsteps * (s + 1) / ksplit) * SK_STEP);
  const int sub = 8 * (lane >> 4);  // this lane's 8 of each 32-wide K piece
  const uint16_t *wp[NW];
#pragma unroll
  for (int j = 0; j < NW; ++j) wp[j] = W + (long)(n0 + 16 * j + (lane & 15)) * K + sub;
  const f16 *ap[RG];
#pragma unroll
  for (int g = 0; g < RG; ++g)
    ap[g] = A + (long)min(g * 16 + (lane & 15), rows - 1) * K * AS + sub;
  f32x4 acc[NW][RG];
#pragma unroll
  for (int j = 0; j < NW; ++j)
#pragma unroll
    for (int g = 0; g < RG; ++g) acc[j][g] = f32x4{0.f, 0.f, 0.f, 0.f};

  for (int k = k0; k < k1; k += SK_STEP) {
    // Every load of the step is issued before the first product; pieces past
    // the slice end (a short last step) re-load its last piece and multiply
    // zero activations (cnt is the same for the whole wave).
    const int cnt = min(SK_U, (k1 - k) / 32);
    u32x4 wv[SK_U][NW], av[SK_U][RG][AS];
#pragma unroll
    for (int u = 0; u < SK_U; ++u) {
      const int kk = k + 32 * min(u, cnt - 1);
#pragma unroll
      for (int j = 0; j < NW; ++j) wv[u][j] = ld16(wp[j] + kk);
#pragma unroll
      for (int g = 0; g < RG; ++g)
#pragma unroll
        for (int h = 0; h < AS; ++h) av[u][g][h] = ld16(ap[g] + h * K + kk);
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int u = 0; u < SK_U; ++u) {
      const u32x4 zero = {0u, 0u, 0u, 0u};
#pragma unroll
      for (int j = 0; j < NW; ++j) {
        const f16x8 wf = as_h8(WCVT ? sk_bf16_to_f16(wv[u][j]) : wv[u][j]);
#pragma unroll
        for (int g = 0; g < RG; ++g)
#pragma unroll
          for (int h = 0; h < AS; ++h)
            acc[j][g] = __builtin_amdgcn_mfma_f32_16x16x32_f16(
                wf, as_h8(u < cnt ? av[u][g][h] : zero), acc[j][g], 0, 0, 0);
      }
    }
  }
  // Lane l holds activation row l % 16 of each group and weight rows
  // n0 + 16 j + 4 (l / 16) + i, i < 4.
  if constexpr (OUT == SK_ARGMAX) {
    __shared__ float bv[4][16 * RG];
    __shared__ int bi[4][16 * RG];
#pragma unroll
    for (int g = 0; g < RG; ++g) {
      float v = acc[0][g][0];
      int vi = n0 + 4 * (lane >> 4);
#pragma unroll
      for (int i = 1; i < 4 * NW; ++i)
        if (acc[i >> 2][g][i & 3] > v) {  // ascending indices: a strict > keeps the lowest
          v = acc[i >> 2][g][i & 3];
          vi = n0 + 16 * (i >> 2) + 4 * (lane >> 4) + (i & 3);
        }
#pragma unroll
      for (int o = 16; o < 64; o <<= 1) {
        const float v2 = __shfl_xor(v, o, 64);
        const int i2 = __shfl_xor(vi, o, 64);
        if (v2 > v || (v2 == v && i2 < vi)) {
          v = v2;
          vi = i2;
        }
      }
      if (lane < 16) {
        bv[w][g * 16 + lane] = v;
        bi[w][g * 16 + lane] = vi;
      }
    }
    __syncthreads();
    const int r = threadIdx.x;
    if (r < 16 * RG && r < rows) {
      float v = bv[0][r];
      int vi = bi[0][r];
#pragma unroll
      for (int i = 1; i < 4; ++i)
        if (bv[i][r] > v) {  // waves hold ascending index ranges
          v = bv[i][r];
          vi = bi[i][r];
        }
      reinterpret_cast<float2 *>(part)[(long)b * rows + r] = make_float2(v, __int_as_float(vi));
    }
  } else if constexpr (OUT == SK_LSE) {
    __shared__ float2 red[4][16 * RG];
#pragma unroll
    for (int g = 0; g < RG; ++g) {
      const int r = g * 16 + (lane & 15);
      const int at = r < rows ? tgt[r] - (n0 + 4 * (lane >> 4)) : -1;
      float m = -INFINITY, sum = 0.f;
#pragma unroll
      for (int i = 0; i < 4 * NW; ++i) {
        if (at == 16 * (i >> 2) + (i & 3)) tgt_logit[r] = acc[i >> 2][g][i & 3];
        m = fmaxf(m, acc[i >> 2][g][i & 3]);
      }
      m = fmaxf(m, __shfl_xor(m, 16, 64));
      m = fmaxf(m, __shfl_xor(m, 32, 64));
#pragma unroll
      for (int i = 0; i < 4 * NW; ++i) {
        const float x = acc[i >> 2][g][i & 3];
        sum += x == -INFINITY ? 0.f : __expf(x - m);
      }
      sum += __shfl_xor(sum, 16, 64);
      sum += __shfl_xor(sum, 32, 64);
      if (lane < 16) red[w][g * 16 + lane] = make_float2(m, sum);
    }
    __syncthreads();
    const int r = threadIdx.x;
    if (r < 16 * RG && r < rows) {
      float m = red[0][r].x;
#pragma unroll
      for (int i = 1; i < 4; ++i) m = fmaxf(m, red[i][r].x);
      float sum = 0.f;
#pragma unroll
      for (int i = 0; i < 4; ++i)
        sum += red[i][r].y == 0.f ? 0.f : red[i][r].y * __expf(red[i][r].x - m);
      reinterpret_cast<float2 *>(part)[(long)b * rows + r] = make_float2(m, sum);
    }
  } else {
#pragma unroll
    for (int g = 0; g < RG; ++g) {
      const int r = g * 16 + (lane & 15);
      if (r < rows)
        *reinterpret_cast<f32x4 *>(part + ((long)s * rows + r) * N + n0 + 4 * (lane >> 4)) =
            acc[0][g];
    }
  }
}

// Block per row: x += sum of the slices; then, if g is given, the RMSNorm of
// the new row into y (fp16, with its remainder half when split == 2).
__global__ __launch_bounds__(1024) void k_skinny_residual(const float *__restrict__ part,
                                                          int ksplit, int rows, int d,
                                                          float *__restrict__ x, const bf16 *g,
                                                          float eps, f16 *__restrict__ y,
                                                          int split) {
  __shared__ float red[16];
  const int r = blockIdx.x, lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  float *xr = x + (long)r * d;
  const long stride = (long)rows * d;
  float ss = 0.f;
  for (int c = threadIdx.x; c < d; c += 1024) {
    const float v = xr[c] + sum_slices(part, ksplit, stride, (long)r * d + c);
    xr[c] = v;
    ss += v * v;
  }
  if (!g) return;
  ss = wave_sum(ss);
  if (lane == 0) red[w] = ss;
  __syncthreads();
  float t = 0.f;
#pragma unroll
  for (int i = 0; i < 16; ++i) t += red[i];
  const float rs = rsqrtf(t / (float)d + eps);
  f16 *yr = y + (long)r * d * split;
  for (int c = threadIdx.x; c < d; c += 1024) {
    const float v = xr[c] * rs * static_cast<float>(g[c]);
    const f16 hi = static_cast<f16>(v);
    yr[c] = hi;
    if (split == 2) yr[d + c] = static_cast<f16>(v - static_cast<float>(hi));
  }
}

// Thread per (row, f): h = silu(gate) * up from the summed slices (gate rows
// 0..F-1, up rows F..2F-1 of the product), fp16 with its remainder half when
// hsplit == 2.
__global__ __launch_bounds__(256) void k_skinny_swiglu(const float *__restrict__ part,
                                                       int ksplit, int rows, int F, int hsplit,
                                                       f16 *__restrict__ h) {
  const long i = (long)blockIdx.x * 256 + threadIdx.x;
  if (i >= (long)rows * F) return;
  const int r = (int)(i / F), f = (int)(i % F);
  const long stride = (long)rows * 2 * F, base = (long)r * 2 * F;
  const float gt = sum_slices(part, ksplit, stride, base + f);
  const float up = sum_slices(part, ksplit, stride, base + F + f);
  const float v = gt / (1.f + __expf(-gt)) * up;
  const f16 hi = static_cast<f16>(v);
  const long o = (long)r * F * hsplit + f;
  h[o] = hi;
  if (hsplit == 2) h[o + F] = static_cast<f16>(v - static_cast<float>(hi));
}

// Thread per (row, head slot, d < 64): rotary + stores of the pair (d, d + 64).
__global__ __launch_bounds__(256) void k_skinny_qkv(const float *__restrict__ part, int ksplit,
                                                    int rows, int n_heads, int n_kv,
                                                    QKVOut<f16> o) {
  const int nslots = n_heads + 2 * n_kv, N = nslots * 128;
  const long i = (long)blockIdx.x * 256 + threadIdx.x;
  if (i >= (long)rows * nslots * 64) return;
  const int r = (int)(i / (nslots * 64)), rem = (int)(i % (nslots * 64));
  const int slot = rem / 64, d = rem % 64;
  const long stride = (long)rows * N, base = (long)r * N + slot * 128 + d;
  const float x1 = sum_slices(part, ksplit, stride, base);
  const float x2 = sum_slices(part, ksplit, stride, base + 64);
  qkv_store(o, n_heads, n_kv, slot, r, d, x1, x2);
}

// ------------------------------------------------- at most 8 rows: one launch
// A projection of at most 8 rows as one launch: the RMSNorm of its input and
// its epilogue included, no partials in memory. What bounds such a launch is
// the time to fill the chip and one or two memory round trips, so everything
// a block needs is asked for at once: 16 waves share a group of 8 weight rows
// and split K evenly, each lane holding all of its 16-byte weight loads (PW)
// before the first product; the waves' sums meet in LDS. The 16 x 16 tile of
// the matrix core holds the even and odd 32-wide pieces of K side by side,
// weight rows 0-7 / 8-15 and activation rows (columns) 0-7 / 8-15 of it, and
// its two diagonal quadrants are added: 2048 outputs are 256 blocks, one per
// CU, and a load covers whole 128-byte lines (the halves of K instead of its
// pieces side by side: 13.5 us against 12.0 for 2048 x 11008).
// A block of the norm forms walks groups blockIdx.x, + gridDim.x, ..., D groups'
// loads in flight; one of the residual form takes one group.
// Decode layer of the 3B drafter, 3 rows: product, reduce and norm launches 63
// us, these four 42 us (QKV 7.4, O 4.6, gate/up 18.2 = 5.0 TB/s, down 11.9 =
// 3.8 TB/s). Tiles of 16 whole rows for 9..16 activation rows were 2% slower
// than those launches.
enum { FEW_QKV, FEW_SWIGLU, FEW_RESIDUAL };
struct FewArgs {
  const f16 *A;      // FEW_RESIDUAL: activations [rows][AS K]
  float *x;          // residual rows: the normed input, or the output
  const bf16 *g;     // gain of the input's norm
  float eps;
  const uint16_t *W;
  int rows, N, K;    // N weight rows
  f16 *h;            // FEW_SWIGLU: [rows][AS N / 2]
  int n_heads, n_kv;
  QKVOut<f16> o;
};

// AS = 2: the activations are fp16 value + remainder (A and h rows [hi | lo]).
template <int EPI, int AS, int PW, int D, bool WCVT, int WPE>
__global__ __launch_bounds__(1024, WPE) void k_few(FewArgs a) {
  constexpr int S = 128 + 4;  // LDS words per wave (+ 4: conflict-free column reads)
  constexpr bool NORM = EPI != FEW_RESIDUAL;
  __shared__ float red[2][16 * S];
  __shared__ float ssq[16][8];
  const int tid = threadIdx.x, lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int half = (lane >> 3) & 1, lr = lane & 7;
  const int hp = a.K / 64;            // pairs of 32-wide pieces
  const int p0 = hp * w / 16, cnt = hp * (w + 1) / 16 - p0;
  const int kbase = half * 32 + 8 * (lane >> 4);
  const int ngroups = a.N / 8;
  // K offset of the wave's pair j past the lane's own kbase (pairs past the
  // slice re-load its last one and take no part in the products).
  const auto koff = [&](int j) { return 64 * min(p0 + max(0, min(j, cnt - 1)), hp - 1); };
  // Buffer loads: the lane's offset once, the pairs' in scalar registers.
  const auto rsrc = [](const void *p, long bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p), (short)0, (int)bytes,
                                             0x00020000);
  };
  const auto ld = [](__amdgpu_buffer_rsrc_t r, uint32_t lane_off, uint32_t off) {
    return __builtin_bit_cast(u32x4,
                              __builtin_amdgcn_raw_buffer_load_b128(r, lane_off, off, 0));
  };
  const __amdgpu_buffer_rsrc_t rw = rsrc(a.W, (long)a.N * a.K * 2);
  const auto wrow = [&](int g) {      // weight row of this lane in group g
    const int up = lr >> 2, i = lr & 3;
    if constexpr (EPI == FEW_QKV)     // dims (d, d + 64) of a head slot
      return (g >> 4) * 128 + (g & 15) * 4 + i + 64 * up;
    else if constexpr (EPI == FEW_SWIGLU)
      return g * 4 + i + up * (a.N / 2);
    else
      return g * 8 + lr;
  };
  const int arow = min(lr, a.rows - 1);

  u32x4 wv[D][PW];
  const auto load_w = [&](int i, int g, int j0) {
    const uint32_t off = ((uint32_t)wrow(min(g, ngroups - 1)) * a.K + kbase) * 2;
#pragma unroll
    for (int j = 0; j < PW; ++j) wv[i][j] = ld(rw, off, 2 * koff(j0 + j));
  };
  const auto load_first = [&] {
#pragma unroll
    for (int i = 0; i < D; ++i) load_w(i, blockIdx.x + i * gridDim.x, 0);
  };
  f16x8 af[PW][AS];
  const auto load_a = [&](int j0) {
    const __amdgpu_buffer_rsrc_t ra = rsrc(a.A, (long)a.rows * a.K * AS * 2);
#pragma unroll
    for (int j = 0; j < PW; ++j)
#pragma unroll
      for (int h = 0; h < AS; ++h)
        af[j][h] = as_h8(ld(ra, (arow * AS * a.K + kbase) * 2, 2 * (koff(j0 + j) + h * a.K)));
  };
  // This thread's output (with its 15 neighbours): activation row r, weight
  // row c of the group (q | k | v and gate / up: member c / 4 of pair c % 4, the
  // members in neighbouring 16-lane rows).
  const int r = tid >> 7, rc = min(r, a.rows - 1), c0 = (tid >> 4) & 7;
  const int c = EPI == FEW_RESIDUAL ? c0 : (c0 >> 1) + 4 * (c0 & 1);
  // What the epilogue needs from memory, asked for before the products (the
  // position before all else: the rotary entries hang on it).
  float xo = 0.f;
  float2 cs = {1.f, 0.f};
  int pos = 0, crow = 0;
  if constexpr (EPI == FEW_QKV) {
    pos = qkv_row_pos(a.o, rc);
    crow = qkv_cache_row(a.o, rc);
  }
  const auto load_cs = [&](int g) { cs = a.o.rope[(long)pos * 64 + (g & 15) * 4 + (c0 >> 1)]; };
  if constexpr (NORM) {
    f32x4 xv[PW][2];
    u32x4 gv[PW];
    const __amdgpu_buffer_rsrc_t rx = rsrc(a.x, (long)a.rows * a.K * 4);
    const __amdgpu_buffer_rsrc_t rg = rsrc(a.g, (long)a.K * 2);
    const uint32_t off = (arow * a.K + kbase) * 4;
#pragma unroll
    for (int j = 0; j < PW; ++j) {
      xv[j][0] = __builtin_bit_cast(f32x4, ld(rx, off, 4 * koff(j)));
      xv[j][1] = __builtin_bit_cast(f32x4, ld(rx, off + 16, 4 * koff(j)));
      gv[j] = ld(rg, kbase * 2, 2 * koff(j));
    }
    __builtin_amdgcn_sched_barrier(0);
    load_first();
    if constexpr (EPI == FEW_QKV) load_cs(blockIdx.x);
    __builtin_amdgcn_sched_barrier(0);
    float ss = 0.f;
#pragma unroll
    for (int j = 0; j < PW; ++j)
      if (j < cnt)
#pragma unroll
        for (int e = 0; e < 8; ++e) ss += xv[j][e >> 2][e & 3] * xv[j][e >> 2][e & 3];
    ss += row_rotated<0x128>(ss);
    auto sw = __builtin_amdgcn_permlane32_swap(__float_as_uint(ss), __float_as_uint(ss), false,
                                               false);
    ss = __uint_as_float(sw[0]) + __uint_as_float(sw[1]);
    sw = __builtin_amdgcn_permlane16_swap(__float_as_uint(ss), __float_as_uint(ss), false, false);
    ss = __uint_as_float(sw[0]) + __uint_as_float(sw[1]);
    if (lane < 8) ssq[w][lane] = ss;
    __syncthreads();
    float t = 0.f;
#pragma unroll
    for (int i = 0; i < 16; ++i) t += ssq[i][lr];
    const float rs = rsqrtf(t / (float)a.K + a.eps);
#pragma unroll
    for (int j = 0; j < PW; ++j)
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const uint32_t gw = gv[j][e >> 1];
        const float gf = __uint_as_float(e & 1 ? gw & 0xFFFF0000u : gw << 16);
        const float v = xv[j][e >> 2][e & 3] * rs * gf;
        const f16 hi = static_cast<f16>(v);
        af[j][0][e] = hi;
        if constexpr (AS == 2) af[j][1][e] = static_cast<f16>(v - static_cast<float>(hi));
      }
  } else {
    load_first();
    load_a(0);
    xo = a.x[(long)rc * a.N + blockIdx.x * 8 + c];
  }

  int buf = 0;
  for (int g0 = blockIdx.x; g0 < ngroups; g0 += D * gridDim.x) {
#pragma unroll
    for (int i = 0; i < D; ++i) {
      const int g = g0 + i * gridDim.x;
      if (g >= ngroups) break;
      f32x4 acc = {0.f, 0.f, 0.f, 0.f};
      for (int j0 = 0;;) {
#pragma unroll
        for (int j = 0; j < PW; ++j)
          if (j0 + j < cnt) {
            const f16x8 wf = as_h8(WCVT ? sk_bf16_to_f16(wv[i][j]) : wv[i][j]);
#pragma unroll
            for (int h = 0; h < AS; ++h)
              acc = __builtin_amdgcn_mfma_f32_16x16x32_f16(wf, af[j][h], acc, 0, 0, 0);
          }
        if (NORM || (j0 += PW) >= cnt) break;
        load_w(i, g, j0);
        load_a(j0);
      }
      if (NORM && g + D * (int)gridDim.x < ngroups) load_w(i, g + D * gridDim.x, 0);
      // Lane: activation row lane % 8, weight rows 4 (lane / 16 % 2) + 0..3 of
      // quadrant (lane / 32, lane / 8 % 2).
      if (half == lane >> 5)
        *reinterpret_cast<f32x4 *>(&red[buf][w * S + half * 64 + lr * 8 + (lane >> 2 & 4)]) = acc;
      __syncthreads();
      const float *p = &red[buf][(tid & 15) * S + r * 8 + c];
      float v = p[0] + p[64];
      v += row_rotated<0x128>(v);
      v += row_rotated<0x124>(v);
      v += row_rotated<0x122>(v);
      v += row_rotated<0x121>(v);
      if constexpr (EPI == FEW_RESIDUAL) {
        if ((tid & 15) == 0 && r < a.rows) a.x[(long)r * a.N + g * 8 + c] = xo + v;
        return;
      }
      float v2 = __shfl_xor(v, 16, 64);
      if ((tid & 31) == 0 && r < a.rows) {
        if constexpr (EPI == FEW_SWIGLU) {
          const int F = a.N / 2;
          const float hv = v / (1.f + __expf(-v)) * v2;
          const f16 hi = static_cast<f16>(hv);
          f16 *hr = a.h + (long)r * F * AS + g * 4 + c;
          *hr = hi;
          if constexpr (AS == 2) hr[F] = static_cast<f16>(hv - static_cast<float>(hi));
        } else {
          const int slot = g >> 4;
          qk_turn(a.o, a.n_heads, a.n_kv, slot, v, v2, cs);
          qkv_store_at(a.o, a.n_heads, a.n_kv, slot, r, (g & 15) * 4 + c, v, v2,
                       [&] { return crow; });
        }
      }
      if (EPI == FEW_QKV && g + (int)gridDim.x < ngroups) load_cs(g + gridDim.x);
      buf ^= 1;
    }
  }
}

template <int EPI, int AS, int PW, int D, int WPE>
hipError_t launch_few(const FewArgs &a, bool w_f16, int most, hipStream_t s) {
  const int blocks = std::min(a.N / 8, most);
  if (w_f16)
    k_few<EPI, AS, PW, D, false, WPE><<<blocks, 1024, 0, s>>>(a);
  else
    k_few<EPI, AS, PW, D, true, WPE><<<blocks, 1024, 0, s>>>(a);
  return hipGetLastError();
}

// Loads per lane of a weight row group.
inline int few_loads(int K) { return (K / 64 + 15) / 16; }

// The gate/up projection keeps two groups' loads in flight on two blocks a CU
// (18.2 us for 22016 x 2048; one group 31.3, three 19.5, four on one block a CU
// 19.2) where the registers allow it; the QKV projection's few groups are one
// block a CU's worth (7.4 us for 2560 x 2048, about 1.3 more with two blocks a CU).
template <int EPI>
hipError_t launch_few_norm(const FewArgs &a, bool w_f16, int asplit, hipStream_t s) {
  constexpr bool GU = EPI == FEW_SWIGLU;
  constexpr int D = GU ? 2 : 1;
  if (few_loads(a.K) <= 2) {
    if (asplit == 2) return launch_few<EPI, 2, 2, D, 4>(a, w_f16, 256, s);
    return launch_few<EPI, 1, 2, D, GU ? 8 : 4>(a, w_f16, GU ? 512 : 256, s);
  }
  return asplit == 2 ? launch_few<EPI, 2, 4, D, 4>(a, w_f16, 256, s)
                     : launch_few<EPI, 1, 4, D, 4>(a, w_f16, 256, s);
}

template <int OUT, int RG, int AS, int NW = 1>
hipError_t launch_rg(const f16 *A, int rows, const void *W, bool w_f16, int N, int K, int ks,
                     float *part, hipStream_t s, const int32_t *tgt, float *tgt_logit) {
  const dim3 grid(N / (SK_ROWS * NW), ks);
  const uint16_t *W16 = static_cast<const uint16_t *>(W);
  if (w_f16)
    k_skinny<RG, AS, false, OUT, NW><<<grid, 256, 0, s>>>(A, rows, W16, N, K, ks, part, tgt,
                                                      tgt_logit);
  else
    k_skinny<RG, AS, true, OUT, NW><<<grid, 256, 0, s>>>(A, rows, W16, N, K, ks, part, tgt,
                                                     tgt_logit);
  return hipGetLastError();
}

hipError_t launch(const f16 *A, int rows, int asplit, const void *W, bool w_f16, int N, int K,
                  int ks, float *part, hipStream_t s) {
  if (rows <= 16)
    return asplit == 2
               ? launch_rg<SK_PART, 1, 2>(A, rows, W, w_f16, N, K, ks, part, s, nullptr, nullptr)
               : launch_rg<SK_PART, 1, 1>(A, rows, W, w_f16, N, K, ks, part, s, nullptr, nullptr);
  return asplit == 2
             ? launch_rg<SK_PART, 2, 2>(A, rows, W, w_f16, N, K, ks, part, s, nullptr, nullptr)
             : launch_rg<SK_PART, 2, 1>(A, rows, W, w_f16, N, K, ks, part, s, nullptr, nullptr);
}

// LM head of few rows (unsplit activations, one K slice).
template <int OUT>
hipError_t launch_lm(const f16 *A, int rows, const void *W, bool w_f16, int vocab, int K,
                     float2 *part, hipStream_t s, const int32_t *tgt, float *tgt_logit) {
  if (rows < 1 || rows > kSkinnyMaxRows || vocab % SK_ROWS || K % 32 || K <= 0)
    return hipErrorInvalidValue;
  float *p = reinterpret_cast<float *>(part);
  constexpr int NW = OUT == SK_LSE ? 2 : 1;
  if (vocab % (SK_ROWS * NW) == 0)
    return rows <= 16
               ? launch_rg<OUT, 1, 1, NW>(A, rows, W, w_f16, vocab, K, 1, p, s, tgt, tgt_logit)
               : launch_rg<OUT, 2, 1, NW>(A, rows, W, w_f16, vocab, K, 1, p, s, tgt, tgt_logit);
  return rows <= 16 ? launch_rg<OUT, 1, 1>(A, rows, W, w_f16, vocab, K, 1, p, s, tgt, tgt_logit)
                    : launch_rg<OUT, 2, 1>(A, rows, W, w_f16, vocab, K, 1, p, s, tgt, tgt_logit);
}

bool skinny_args_ok(int rows, int N, int K, int asplit) {
  return rows >= 1 && rows <= kSkinnyMaxRows && N % SK_ROWS == 0 && K % 32 == 0 && K > 0 &&
         (asplit == 1 || asplit == 2);
}

}  // namespace

int skinny_split(int N, int K) {
  const int blocks = std::max(1, N / SK_ROWS);
  const int by_k = (K + SK_STEP - 1) / SK_STEP;
  return std::min({by_k, std::max(1, (1024 + blocks - 1) / blocks), kSkinnyMaxSplit});
}

size_t skinny_part_floats(int rows, int N, int K) {
  return (size_t)skinny_split(N, K) * rows * N;
}

hipError_t skinny_residual(const f16 *A, int rows, int asplit, const void *W, bool w_f16, int N,
                           int K, float *x, const bf16 *g, float eps, f16 *y, int ysplit,
                           float *part, hipStream_t s) {
  if (rows == 0) return hipSuccess;
  if (!skinny_args_ok(rows, N, K, asplit)) return hipErrorInvalidValue;
  const int ks = skinny_split(N, K);
  hipError_t e = launch(A, rows, asplit, W, w_f16, N, K, ks, part, s);
  if (e != hipSuccess) return e;
  k_skinny_residual<<<rows, 1024, 0, s>>>(part, ks, rows, N, x, g, eps, y, ysplit);
  return hipGetLastError();
}

hipError_t skinny_swiglu(const f16 *A, int rows, int asplit, const void *W, bool w_f16, int F,
                         int K, f16 *h, float *part, hipStream_t s) {
  if (rows == 0) return hipSuccess;
  if (!skinny_args_ok(rows, 2 * F, K, asplit)) return hipErrorInvalidValue;
  const int ks = skinny_split(2 * F, K);
  hipError_t e = launch(A, rows, asplit, W, w_f16, 2 * F, K, ks, part, s);
  if (e != hipSuccess) return e;
  const long n = (long)rows * F;
  k_skinny_swiglu<<<(unsigned)((n + 255) / 256), 256, 0, s>>>(part, ks, rows, F, asplit, h);
  return hipGetLastError();
}

hipError_t skinny_qkv_rope(const f16 *A, int rows, int asplit, const void *W, bool w_f16, int K,
                           int n_heads, int n_kv, const QKVOut<f16> &out, float *part,
                           hipStream_t s) {
  if (rows == 0) return hipSuccess;
  const int N = (n_heads + 2 * n_kv) * 128;
  if (!skinny_args_ok(rows, N, K, asplit)) return hipErrorInvalidValue;
  const int ks = skinny_split(N, K);
  hipError_t e = launch(A, rows, asplit, W, w_f16, N, K, ks, part, s);
  if (e != hipSuccess) return e;
  const long n = (long)rows * (n_heads + 2 * n_kv) * 64;
  k_skinny_qkv<<<(unsigned)((n + 255) / 256), 256, 0, s>>>(part, ks, rows, n_heads, n_kv, out);
  return hipGetLastError();
}

bool few_ok(int rows, int d, int att, int F) {
  // (The norm forms hold a wave's share of K in registers: 4 loads a lane. The
  // residual forms take any K of whole 64s. Weight offsets are 32 bits.)
  return rows >= 1 && rows <= 8 && d % 64 == 0 && few_loads(d) <= 4 && att % 64 == 0 &&
         F % 64 == 0 && (size_t)std::max(2 * F, 3 * att) * d * 2 <= UINT32_MAX;
}

hipError_t few_qkv_rope(const float *x, const bf16 *g, float eps, int rows, int asplit,
                        const void *W, bool w_f16, int K, int n_heads, int n_kv,
                        const QKVOut<f16> &out, hipStream_t s) {
  const FewArgs a{nullptr, const_cast<float *>(x), g, eps, static_cast<const uint16_t *>(W), rows,
                  (n_heads + 2 * n_kv) * 128, K, nullptr, n_heads, n_kv, out};
  return launch_few_norm<FEW_QKV>(a, w_f16, asplit, s);
}

hipError_t few_swiglu(const float *x, const bf16 *g, float eps, int rows, int asplit,
                      const void *W, bool w_f16, int F, int K, f16 *h, hipStream_t s) {
  const FewArgs a{nullptr, const_cast<float *>(x), g, eps, static_cast<const uint16_t *>(W), rows,
                  2 * F, K, h, 0, 0, {}};
  return launch_few_norm<FEW_SWIGLU>(a, w_f16, asplit, s);
}

hipError_t few_residual(const f16 *A, int rows, int asplit, const void *W, bool w_f16, int N,
                        int K, float *x, hipStream_t s) {
  const FewArgs a{A, x, nullptr, 0.f, static_cast<const uint16_t *>(W), rows, N, K, nullptr, 0, 0,
                  {}};
  constexpr int EPI = FEW_RESIDUAL, ALL = INT32_MAX;
  const int loads = few_loads(K);
  if (loads <= 2)
    return asplit == 2 ? launch_few<EPI, 2, 2, 1, 8>(a, w_f16, ALL, s)
                       : launch_few<EPI, 1, 2, 1, 8>(a, w_f16, ALL, s);
  if (asplit == 2) return launch_few<EPI, 2, 6, 1, 4>(a, w_f16, ALL, s);
  // More groups than CUs: two blocks a CU with fewer loads each.
  if (loads <= 6 || N / 8 > 256) return launch_few<EPI, 1, 6, 1, 8>(a, w_f16, ALL, s);
  return launch_few<EPI, 1, 11, 1, 4>(a, w_f16, ALL, s);
}

int skinny_lm_chunks(int vocab) { return vocab % SK_ROWS ? 0 : vocab / SK_ROWS; }

int skinny_lse_chunks(int vocab) {
  return vocab % (2 * SK_ROWS) == 0 ? vocab / (2 * SK_ROWS) : skinny_lm_chunks(vocab);
}

// Each row costs the stream its loads and products, more the wider the rows,
// and the merge twice the tiles' chunks; a tile of up to 128 rows costs the same
// for all of them. Head and merge of a 152k vocabulary, us: they cross past 32
// rows at K 2048 (183 against 195 at 32), at 19 / 26 / 25 / 20 rows for K 2560 / 3072 /
// 3584 / 4096, at 15 / 17 for 5120 / 8192 with fp16 weights (24 rows of 5120: 430
// against 401), and at 21 to 28 with bf16 ones, where the tiles cost more. One
// line for both, so that they score alike.
int skinny_lse_rows(int K) { return K <= 2048 ? 32 : K <= 4096 ? 24 : 16; }

hipError_t skinny_lmargmax(const f16 *A, int rows, const void *W, bool w_f16, int vocab, int K,
                           float2 *part, hipStream_t s) {
  if (rows == 0) return hipSuccess;
  return launch_lm<SK_ARGMAX>(A, rows, W, w_f16, vocab, K, part, s, nullptr, nullptr);
}

hipError_t skinny_lmhead(const f16 *A, int rows, const void *W, bool w_f16, int vocab, int K,
                         const int32_t *lm_tgt, float2 *part, float *tgt_logit, hipStream_t s) {
  if (rows == 0) return hipSuccess;
  return launch_lm<SK_LSE>(A, rows, W, w_f16, vocab, K, part, s, lm_tgt, tgt_logit);
}

}  // namespace vsr
