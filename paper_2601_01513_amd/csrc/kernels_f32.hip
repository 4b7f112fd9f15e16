// Kernels of the fp32 contexts: projections with fused RMSNorm and epilogues,
// attention, LM head. fp32 operands and fp32 accumulation throughout, on the
// fp32 matrix instruction v_mfma_f32_16x16x4_f32. The shapes of these contexts
// are small, so a pass is bound by launches and by the latency inside each
// launch, not by arithmetic: every kernel spreads one output tile's
// contraction (or key range) over the waves of a block, loads its operands
// straight from global memory (L2) into the registers the matrix instruction
// reads, and does in one launch what it can.
//
// Operand loads: for a 16-wide piece of the contraction lane l loads the four
// consecutive values 4 (l / 16) .. + 3 of row l % 16; product j of the four
// takes component j of both operands, i.e. contraction index 4 (l / 16) + j in
// lane group l / 16, the same index for both.
// Result layout: lane l, register r: row 4 (l / 16) + r, column l % 16.
#include <algorithm>

#include "common.h"

namespace vsr {

namespace {

__device__ __forceinline__ float silu_f(float g) { return g / (1.f + __expf(-g)); }

__device__ __forceinline__ f32x4 mfma4(f32x4 a, f32x4 b, f32x4 c) {
#pragma unroll
  for (int j = 0; j < 4; ++j) c = __builtin_amdgcn_mfma_f32_16x16x4f32(a[j], b[j], c, 0, 0, 0);
  return c;
}

// Four consecutive values p[k .. k+3] of a row of n values; FAST: the row is
// 16-byte aligned and n a multiple of 16, otherwise element by element with
// zeros past the end.
template <bool FAST>
__device__ __forceinline__ f32x4 ld4(const float *p, int k, int n) {
  if constexpr (FAST) {
    return *reinterpret_cast<const f32x4 *>(p + k);
  } else {
    f32x4 v;
#pragma unroll
    for (int j = 0; j < 4; ++j) v[j] = k + j < n ? p[k + j] : 0.f;
    return v;
  }
}

// ------------------------------------------------------------------ products
// C = f(A) . W^T for A [rows][K], W [.][K]. A block owns 16 MG rows and NG
// groups of 16 weight rows; its four waves take the 16-wide pieces of K in
// turn (wave w pieces w, w + 4, ...: together they read whole cache lines)
// and add their partial products through LDS in wave order, so a result does
// not depend on the grid or on the row's place in it.
// NORM: f(A) = RMSNorm(A) g: the products take A * g, the waves sum the rows'
// squares beside them and the epilogue scales the row (no norm launch; each
// of these contexts' norms cost about 4.6 us of a pass).
// The tiny model's QKV projection (384 prefix + candidate rows, K 256, 768
// columns): 9.7 us; with one thread per output and separate norms and passes
// it took 196 + 57 + 9 us. Its whole verify pass: 2889 -> 101 us.
enum { EPI_QKV, EPI_RESIDUAL, EPI_SWIGLU, EPI_LSE, EPI_ARGMAX };

struct F32Gemm {
  const float *A, *W;
  int rows, K, n;  // n: rotary pairs (QKV), F (SwiGLU), or rows of W
  int nrt, ct0;    // row tiles: block b is row tile b % nrt, column tile ct0 + b / nrt
  const float *g;
  float eps;
  const int32_t *row_lo;  // not NULL: row t is h_last if row_lo[t] == t, else A[t - 1]
  const float *h_last;
  int n_heads, n_kv, hd;  // QKV
  QKVOut<float> o;
  float *y;  // residual stream (added to) or FFN hidden
  const int32_t *tgt;
  float2 *part;
  float *tgt_logit;
};

// One rotary pair (dims i, i + hd / 2 of head slot `slot`) of row `row`.
__device__ __forceinline__ void qkv_store_f32(const F32Gemm &a, int row, int pair, float x1,
                                              float x2) {
  const QKVOut<float> &o = a.o;
  const int half = a.hd / 2, slot = pair / half, i = pair % half;
  const bool second = row >= o.split;
  const int row2 = row - o.split;
  if (slot < a.n_heads + a.n_kv) {
    const int pos = second ? o.row_pos2[row2] : o.row_pos ? o.row_pos[row] : row;
    const float2 cs = o.rope[(long)pos * half + i];
    const float y1 = x1 * cs.x - x2 * cs.y, y2 = x2 * cs.x + x1 * cs.y;
    x1 = y1;
    x2 = y2;
  }
  if (slot < a.n_heads) {
    float *q = o.q + ((long)row * a.n_heads + slot) * a.hd;
    q[i] = x1;
    q[i + half] = x2;
    return;
  }
  const int crow = second ? row2 : o.cache_row ? o.cache_row[row] : row;
  const int npos = second ? o.kv_npos2 : o.kv_npos;
  if (slot < a.n_heads + a.n_kv) {
    float *k = (second ? o.k2 : o.k) + ((long)(slot - a.n_heads) * npos + crow) * a.hd;
    k[i] = x1;
    k[i + half] = x2;
  } else {
    float *vt = (second ? o.vt2 : o.vt) + (long)(slot - a.n_heads - a.n_kv) * a.hd * npos + crow;
    vt[(long)i * npos] = x1;
    vt[(long)(i + half) * npos] = x2;
  }
}

template <int EPI, int MG, int NG, bool NORM, bool FAST>
__global__ __launch_bounds__(256) void k_f32_gemm(F32Gemm a) {
  constexpr bool PAIRED = EPI == EPI_QKV || EPI == EPI_SWIGLU;
  constexpr int COLS = PAIRED ? 8 * NG : 16 * NG;  // units of n per block
  constexpr int U = MG * NG > 4 ? 2 : 4;           // pieces per load batch
  __shared__ float red[4][MG * NG][256];
  __shared__ float ssq[4][MG * 16];
  const int t = threadIdx.x, lane = t & 63, w = t >> 6, c16 = lane & 15, sub = 4 * (lane >> 4);
  const int ct = a.ct0 + blockIdx.x / a.nrt;
  const int m0 = (blockIdx.x % a.nrt) * 16 * MG, u0 = ct * COLS;
  const int K = a.K;
  const float *ap[MG], *wp[NG];
#pragma unroll
  for (int i = 0; i < MG; ++i) {
    const int row = min(m0 + 16 * i + c16, a.rows - 1);
    if (a.row_lo)
      ap[i] = a.row_lo[row] == row ? a.h_last : a.A + (long)(row - 1) * K;
    else
      ap[i] = a.A + (long)row * K;
  }
#pragma unroll
  for (int j = 0; j < NG; ++j) {
    long r;
    if constexpr (PAIRED) {
      const int u = min(u0 + 16 * (j >> 1) + c16, a.n - 1);
      if constexpr (EPI == EPI_QKV) {
        const int half = a.hd / 2;
        r = (long)(u / half) * a.hd + u % half + (j & 1) * half;
      } else {
        r = (long)u + (j & 1) * (long)a.n;
      }
    } else {
      r = min(u0 + 16 * j + c16, a.n - 1);
    }
    wp[j] = a.W + r * K;
  }
  f32x4 acc[MG][NG];
  float ss[MG];
#pragma unroll
  for (int i = 0; i < MG; ++i) {
    ss[i] = 0.f;
#pragma unroll
    for (int j = 0; j < NG; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  }
  const int np = (K + 15) / 16;  // pieces of K
  struct Batch {
    f32x4 a[U][MG], w[U][NG], g[U];
  };
  // Pieces p, p + 4, ... of the batch (past the end: the last one again, unused).
  auto load = [&](int p, Batch &b) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int k = 16 * min(p + 4 * u, np - 1) + sub;
#pragma unroll
      for (int i = 0; i < MG; ++i) b.a[u][i] = ld4<FAST>(ap[i], k, K);
#pragma unroll
      for (int j = 0; j < NG; ++j) b.w[u][j] = ld4<FAST>(wp[j], k, K);
      if constexpr (NORM) b.g[u] = ld4<FAST>(a.g, k, K);
    }
  };
  auto step = [&](int p, const Batch &b) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (p + 4 * u >= np) break;
#pragma unroll
      for (int i = 0; i < MG; ++i) {
        f32x4 x = b.a[u][i];
        if constexpr (NORM) {
          ss[i] += x[0] * x[0] + x[1] * x[1] + x[2] * x[2] + x[3] * x[3];
          x *= b.g[u];
        }
#pragma unroll
        for (int j = 0; j < NG; ++j) acc[i][j] = mfma4(x, b.w[u][j], acc[i][j]);
      }
    }
  };
  if (w < np) {
    Batch b0, b1;
    load(w, b0);
    for (int p = w; p < np; p += 8 * U) {
      if (p + 4 * U < np) load(p + 4 * U, b1);
      __builtin_amdgcn_sched_barrier(0);
      step(p, b0);
      if (p + 4 * U >= np) break;
      if (p + 8 * U < np) load(p + 8 * U, b0);
      __builtin_amdgcn_sched_barrier(0);
      step(p + 4 * U, b1);
    }
  }
#pragma unroll
  for (int i = 0; i < MG; ++i) {
#pragma unroll
    for (int j = 0; j < NG; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r) red[w][i * NG + j][64 * r + lane] = acc[i][j][r];
    if constexpr (NORM) {
      float s = ss[i];
      s += __shfl_xor(s, 16, 64);
      s += __shfl_xor(s, 32, 64);
      if (lane < 16) ssq[w][16 * i + lane] = s;
    }
  }
  __syncthreads();
  // Thread t holds row 4 ((t % 64) / 16) + t / 64 of each row group, column
  // t % 16 of each column group.
#pragma unroll
  for (int i = 0; i < MG; ++i) {
    const int lr = 16 * i + 4 * (lane >> 4) + w, row = m0 + lr;
    float v[NG];
#pragma unroll
    for (int j = 0; j < NG; ++j) {
      const int e = i * NG + j;
      v[j] = (red[0][e][t] + red[1][e][t]) + (red[2][e][t] + red[3][e][t]);
    }
    if constexpr (NORM) {
      const float s = (ssq[0][lr] + ssq[1][lr]) + (ssq[2][lr] + ssq[3][lr]);
      const float rs = rsqrtf(s / (float)K + a.eps);
#pragma unroll
      for (int j = 0; j < NG; ++j) v[j] *= rs;
    }
    if constexpr (EPI == EPI_QKV || EPI == EPI_SWIGLU) {
#pragma unroll
      for (int j = 0; j < NG; j += 2) {
        const int u = u0 + 8 * j + c16;
        if (row >= a.rows || u >= a.n) continue;
        if constexpr (EPI == EPI_QKV)
          qkv_store_f32(a, row, u, v[j], v[j + 1]);
        else
          a.y[(long)row * a.n + u] = silu_f(v[j]) * v[j + 1];
      }
    } else if constexpr (EPI == EPI_RESIDUAL) {
#pragma unroll
      for (int j = 0; j < NG; ++j) {
        const int col = u0 + 16 * j + c16;
        if (row < a.rows && col < a.n) a.y[(long)row * a.n + col] += v[j];
      }
    } else if constexpr (EPI == EPI_LSE) {
      // The 16 lanes of a row hold its 16 NG logits of this chunk.
      const int tg = row < a.rows ? a.tgt[row] : -1;
      float m = -INFINITY;
#pragma unroll
      for (int j = 0; j < NG; ++j) {
        const int col = u0 + 16 * j + c16;
        if (col == tg) a.tgt_logit[row] = v[j];
        if (col >= a.n) v[j] = -INFINITY;
        m = fmaxf(m, v[j]);
      }
#pragma unroll
      for (int o = 1; o < 16; o <<= 1) m = fmaxf(m, __shfl_xor(m, o, 64));
      float s = 0.f;
#pragma unroll
      for (int j = 0; j < NG; ++j) s += v[j] == -INFINITY ? 0.f : __expf(v[j] - m);
#pragma unroll
      for (int o = 1; o < 16; o <<= 1) s += __shfl_xor(s, o, 64);
      if (c16 == 0 && row < a.rows) a.part[(long)ct * a.rows + row] = make_float2(m, s);
    } else {
      float best = v[0];
      int bi = u0 + c16 < a.n ? u0 + c16 : -1;
#pragma unroll
      for (int j = 1; j < NG; ++j) {
        const int col = u0 + 16 * j + c16;
        if (col < a.n && v[j] > best) {
          best = v[j];
          bi = col;
        }
      }
#pragma unroll
      for (int o = 1; o < 16; o <<= 1) {
        const float v2 = __shfl_xor(best, o, 64);
        const int i2 = __shfl_xor(bi, o, 64);
        if (i2 >= 0 && (bi < 0 || v2 > best || (v2 == best && i2 < bi))) {
          best = v2;
          bi = i2;
        }
      }
      if (c16 == 0 && row < a.rows)
        a.part[(long)ct * a.rows + row] = make_float2(best, __int_as_float(bi));
    }
  }
}

bool aligned16(const void *p) { return (reinterpret_cast<uintptr_t>(p) & 15) == 0; }

template <int EPI, int MG, int NG, bool NORM>
hipError_t launch_tile(F32Gemm a, hipStream_t s) {
  constexpr int COLS = EPI == EPI_QKV || EPI == EPI_SWIGLU ? 8 * NG : 16 * NG;
  a.nrt = (a.rows + 16 * MG - 1) / (16 * MG);
  const int nct = (a.n + COLS - 1) / COLS;
  // The threads of a launch stay below 2^32 (113k scored rows of a 152k
  // vocabulary reach it): further column tiles take further launches.
  const int per = std::max(1, (1 << 23) / a.nrt);
  // 16-byte loads need aligned rows; other widths and bases load by element.
  const bool fast = a.K % 16 == 0 && aligned16(a.A) && aligned16(a.W) &&
                    (!NORM || aligned16(a.g)) && (!a.row_lo || aligned16(a.h_last));
  for (a.ct0 = 0; a.ct0 < nct; a.ct0 += per) {
    const unsigned grid = (unsigned)a.nrt * std::min(per, nct - a.ct0);
    if (fast)
      k_f32_gemm<EPI, MG, NG, NORM, true><<<grid, 256, 0, s>>>(a);
    else
      k_f32_gemm<EPI, MG, NG, NORM, false><<<grid, 256, 0, s>>>(a);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

// Tile rule: 32 rows x 64 weight rows (16 FLOP per operand byte) once that
// gives four blocks per CU; below it 16 x 32 tiles, four times the blocks. The
// vocabulary epilogues keep 64 columns (their chunk) and choose the rows.
template <int EPI, bool NORM>
hipError_t launch_f32(const F32Gemm &a, hipStream_t s) {
  if (a.rows == 0) return hipSuccess;
  constexpr bool VOCAB = EPI == EPI_LSE || EPI == EPI_ARGMAX;
  constexpr int big = EPI == EPI_QKV || EPI == EPI_SWIGLU ? 32 : 64;
  const long tiles = (long)((a.rows + 31) / 32) * ((a.n + big - 1) / big);
  if (tiles >= 1024) return launch_tile<EPI, 2, 4, NORM>(a, s);
  return launch_tile<EPI, 1, VOCAB ? 4 : 2, NORM>(a, s);
}

// ----------------------------------------------------------------- attention
// Block: 16 query rows of one head, NW waves over 32-key tiles in turn
// (prefix keys, then branch keys), each with an online softmax of its own,
// merged through LDS in wave order. S^T = K . Q^T leaves lane l the scores of
// query l % 16 for keys 4 (l / 16) + r, which is the operand layout of
// O^T = V^T . P^T, so the probabilities go from one product to the next in
// registers. DT: 16-wide pieces of the head dimension. A tile's loads are all
// issued before its first product; tiles no query of the block sees are
// skipped. A tile that some query sees only in part may hold values of rows
// the query must not depend on (a NaN there times a probability of 0 would
// reach it): if such a tile holds a non-finite value its keys are added one by
// one, to the queries that see them.
// 256 prefix + 128 candidate rows of 4 heads (the tiny model): 10.2 us in one
// launch against 180 + 170 us with a wave per row and a key at a time.
template <int DT, int NW, bool FAST>
__global__ __launch_bounds__(64 * NW) void k_f32_attn(F32AttnArgs a) {
  __shared__ float sm[NW][16], sl[NW][16];
  __shared__ float so[NW][DT][256];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, c16 = lane & 15, sub = 4 * (lane >> 4);
  const int h = blockIdx.y, hd = a.hd, kvh = h / (a.n_heads / a.n_kv);
  const int tq0 = a.t0 + blockIdx.x * 16, tq = min(tq0 + c16, a.T - 1);
  const float scale = rsqrtf((float)hd);
  // Visible keys of this lane's query: prefix 0 .. hp, branch blo .. bhi.
  int hp = tq, blo = 0x7fffffff, bhi = -1;
  if (tq >= a.split) {
    const int b = tq - a.split;
    hp = a.P - 1;
    blo = a.row_lo[b];
    bhi = a.q_pos ? a.q_pos[b] : b;
  }
  int hpm = hp, lom = blo, him = bhi;
#pragma unroll
  for (int o = 1; o < 16; o <<= 1) {
    hpm = max(hpm, __shfl_xor(hpm, o, 64));
    lom = min(lom, __shfl_xor(lom, o, 64));
    him = max(him, __shfl_xor(him, o, 64));
  }
  hpm = __builtin_amdgcn_readfirstlane(hpm);
  lom = __builtin_amdgcn_readfirstlane(lom);
  him = __builtin_amdgcn_readfirstlane(him);
  const int np = hpm / 32 + 1, b0 = lom / 32, nb = him >= 0 ? him / 32 - b0 + 1 : 0;

  const float *qr = a.q + ((long)tq * a.n_heads + h) * hd;
  f32x4 q[DT], acc[DT];
#pragma unroll
  for (int d = 0; d < DT; ++d) {
    q[d] = f32x4{0.f, 0.f, 0.f, 0.f};
    if (!FAST || 16 * d + sub < hd) q[d] = ld4<FAST>(qr, 16 * d + sub, hd);
    acc[d] = f32x4{0.f, 0.f, 0.f, 0.f};
  }
  float m = -INFINITY, l = 0.f;
  for (int i = w; i < np + nb; i += NW) {
    const bool pre = i < np;
    const int key0 = 32 * (pre ? i : b0 + i - np);
    const int lo = pre ? 0 : blo, hi = pre ? hp : bhi;
    if (!__any(lo <= key0 + 31 && hi >= key0)) continue;
    const int npos = pre ? a.kv_npos : a.bk_npos;
    const float *kb = (pre ? a.k : a.bk) + (long)kvh * npos * hd;
    const float *vb = (pre ? a.vt : a.bvt) + (long)kvh * npos * hd;
    f32x4 kk[2][DT], vv[2][DT];
#pragma unroll
    for (int s = 0; s < 2; ++s)
#pragma unroll
      for (int d = 0; d < DT; ++d) {
        kk[s][d] = f32x4{0.f, 0.f, 0.f, 0.f};
        if (!FAST || 16 * d + sub < hd)
          kk[s][d] = ld4<FAST>(kb + (long)(key0 + 16 * s + c16) * hd, 16 * d + sub, hd);
      }
#pragma unroll
    for (int s = 0; s < 2; ++s)
#pragma unroll
      for (int d = 0; d < DT; ++d)  // rows past the head repeat the last one (not stored)
        vv[s][d] = *reinterpret_cast<const f32x4 *>(vb + (long)min(16 * d + c16, hd - 1) * npos +
                                                    key0 + 16 * s + sub);
    f32x4 sc[2];
    bool ok[2][4];
    float mx = -INFINITY;
#pragma unroll
    for (int s = 0; s < 2; ++s) {
      sc[s] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int d = 0; d < DT; ++d) sc[s] = mfma4(kk[s][d], q[d], sc[s]);
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int key = key0 + 16 * s + sub + r;
        ok[s][r] = key >= lo && key <= hi;
        sc[s][r] *= scale;
        if (ok[s][r]) mx = fmaxf(mx, sc[s][r]);
      }
    }
    mx = fmaxf(mx, __shfl_xor(mx, 16, 64));
    mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
    const float mn = fmaxf(m, mx), ms = mn == -INFINITY ? 0.f : mn;
    const float alpha = __expf(m - ms);
    m = mn;
    l *= alpha;
#pragma unroll
    for (int s = 0; s < 2; ++s)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        sc[s][r] = ok[s][r] ? __expf(sc[s][r] - ms) : 0.f;
        l += sc[s][r];
      }
    if (__any(alpha != 1.f)) {
#pragma unroll
      for (int d = 0; d < DT; ++d) acc[d] *= alpha;
    }
    bool by_key = false;
    if (!__all(lo <= key0 && hi >= key0 + 31)) {
      bool bad = false;
#pragma unroll
      for (int s = 0; s < 2; ++s)
#pragma unroll
        for (int d = 0; d < DT; ++d)
#pragma unroll
          for (int r = 0; r < 4; ++r) bad |= !isfinite(vv[s][d][r]);
      by_key = __any(bad);
    }
    if (!by_key) {
#pragma unroll
      for (int s = 0; s < 2; ++s)
#pragma unroll
        for (int d = 0; d < DT; ++d) acc[d] = mfma4(vv[s][d], sc[s], acc[d]);
    } else {
      for (int kx = 0; kx < 32; ++kx) {
        const bool mine = sub == 4 * ((kx & 15) >> 2), sees = key0 + kx >= lo && key0 + kx <= hi;
#pragma unroll
        for (int d = 0; d < DT; ++d) {
          float va = 0.f, pb = 0.f;
#pragma unroll
          for (int s = 0; s < 2; ++s)
#pragma unroll
            for (int r = 0; r < 4; ++r)
              if (mine && (kx >> 4) == s && (kx & 3) == r) {
                va = vv[s][d][r];
                pb = sc[s][r];
              }
          const f32x4 z = {0.f, 0.f, 0.f, 0.f};
          const f32x4 add = __builtin_amdgcn_mfma_f32_16x16x4f32(va, pb, z, 0, 0, 0);
          if (sees) acc[d] += add;
        }
      }
    }
  }
  l += __shfl_xor(l, 16, 64);
  l += __shfl_xor(l, 32, 64);
  if (lane < 16) {
    sm[w][lane] = m;
    sl[w][lane] = l;
  }
#pragma unroll
  for (int d = 0; d < DT; ++d)
#pragma unroll
    for (int r = 0; r < 4; ++r) so[w][d][64 * r + lane] = acc[d][r];
  __syncthreads();
  for (int e = threadIdx.x; e < DT * 64; e += 64 * NW) {
    const int d = e >> 6, ln = e & 63, qi = ln & 15, dim = 16 * d + 4 * (ln >> 4);
    if (tq0 + qi >= a.T || dim >= hd) continue;
    float mm = sm[0][qi];
#pragma unroll
    for (int i = 1; i < NW; ++i) mm = fmaxf(mm, sm[i][qi]);
    float ls = 0.f;
    f32x4 o = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int i = 0; i < NW; ++i) {
      const float f = sm[i][qi] == -INFINITY ? (sl[i][qi] == 0.f ? 0.f : 1.f)
                                             : __expf(sm[i][qi] - mm);
      ls += sl[i][qi] * f;
#pragma unroll
      for (int r = 0; r < 4; ++r) o[r] += so[i][d][64 * r + ln] * f;
    }
    const float inv = 1.f / ls;
    float *dst = a.out + ((long)(tq0 + qi) * a.n_heads + h) * hd + dim;
#pragma unroll
    for (int r = 0; r < 4; ++r)
      if (dim + r < hd) dst[r] = o[r] * inv;
  }
}

}  // namespace

hipError_t f32_qkv_rope(const float *x, const float *g, float eps, const float *W, int rows,
                        int K, int n_heads, int n_kv, int hd, const QKVOut<float> &out,
                        hipStream_t s) {
  F32Gemm a{};
  a.A = x;
  a.W = W;
  a.rows = rows;
  a.K = K;
  a.n = (n_heads + 2 * n_kv) * (hd / 2);
  a.g = g;
  a.eps = eps;
  a.n_heads = n_heads;
  a.n_kv = n_kv;
  a.hd = hd;
  a.o = out;
  return launch_f32<EPI_QKV, true>(a, s);
}

hipError_t f32_residual(const float *A, const float *W, int rows, int N, int K, float *x,
                        hipStream_t s) {
  F32Gemm a{};
  a.A = A;
  a.W = W;
  a.rows = rows;
  a.K = K;
  a.n = N;
  a.y = x;
  return launch_f32<EPI_RESIDUAL, false>(a, s);
}

hipError_t f32_swiglu(const float *x, const float *g, float eps, const float *W, int rows, int F,
                      int K, float *h, hipStream_t s) {
  F32Gemm a{};
  a.A = x;
  a.W = W;
  a.rows = rows;
  a.K = K;
  a.n = F;
  a.g = g;
  a.eps = eps;
  a.y = h;
  return launch_f32<EPI_SWIGLU, true>(a, s);
}

int f32_lm_chunks(int vocab) { return (vocab + 63) / 64; }

hipError_t f32_lmhead(const float *A, const float *g, float eps, const int32_t *row_lo,
                      const float *h_last, const float *W, int rows, int vocab, int K,
                      const int32_t *lm_tgt, float2 *part, float *tgt_logit, hipStream_t s) {
  F32Gemm a{};
  a.A = A;
  a.W = W;
  a.rows = rows;
  a.K = K;
  a.n = vocab;
  a.g = g;
  a.eps = eps;
  a.row_lo = row_lo;
  a.h_last = h_last;
  a.tgt = lm_tgt;
  a.part = part;
  a.tgt_logit = tgt_logit;
  return g ? launch_f32<EPI_LSE, true>(a, s) : launch_f32<EPI_LSE, false>(a, s);
}

hipError_t f32_lmargmax(const float *A, const float *W, int rows, int vocab, int K, float2 *part,
                        hipStream_t s) {
  F32Gemm a{};
  a.A = A;
  a.W = W;
  a.rows = rows;
  a.K = K;
  a.n = vocab;
  a.part = part;
  return launch_f32<EPI_ARGMAX, false>(a, s);
}

hipError_t f32_attn(const F32AttnArgs &a, hipStream_t s) {
  if (a.T <= a.t0) return hipSuccess;
  const dim3 grid((a.T - a.t0 + 15) / 16, a.n_heads);
  const bool fast = a.hd % 4 == 0;  // rows of q, k and the output 16-byte aligned
  if (a.hd <= 64)
    fast ? k_f32_attn<4, 8, true><<<grid, 512, 0, s>>>(a)
         : k_f32_attn<4, 8, false><<<grid, 512, 0, s>>>(a);
  else if (a.hd <= 128)
    fast ? k_f32_attn<8, 4, true><<<grid, 256, 0, s>>>(a)
         : k_f32_attn<8, 4, false><<<grid, 256, 0, s>>>(a);
  else
    fast ? k_f32_attn<16, 2, true><<<grid, 128, 0, s>>>(a)
         : k_f32_attn<16, 2, false><<<grid, 128, 0, s>>>(a);
  return hipGetLastError();
}

}  // namespace vsr
