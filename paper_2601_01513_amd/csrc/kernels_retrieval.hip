// Retrieval stage of VideoSpeculateRAG (Section 3.1, Eq. 1-3): keyframes by
// colour-histogram intersection of neighbouring frames, then per-keyframe
// top-k documents by the cosine of CLIP embeddings and the merged top-K.
//
// Every decision is integer or uses one fixed reduction order, so repeated
// calls give identical results: histogram counts are integer LDS atomics;
// the keyframe test compares an integer sum with theta * 3HW in float64;
// rankings break ties by the lower document index.
#include <algorithm>
#include <mutex>

#include "common.h"

namespace vsr {

namespace {

constexpr int BINS = 64;            // per channel, bin = value >> 2
constexpr int HB = 3 * BINS;        // bins of one frame
constexpr int HIST_T = 1024;        // threads of the histogram block

__global__ void k_zero_i32(int32_t *p, long n) {
  const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = 0;
}

// Block (f, part): the histogram of part `part` of `split` of frame f. The
// counts are LDS atomics; the pixels of a scene fall into few bins, so with
// one copy of the histogram per wave most lanes of an atomic met in the same
// word and the copies' serialization bounded the kernel (37 us for 220 frames
// of 336 x 336, 2.0 TB/s). Here every bin has 64 words, one per lane and one
// per LDS bank: lane l counts bin b at word 64 b + l, no two lanes of an
// instruction share a bank, and all waves of the block share the copies.
// Now 19.7 us (3.8 TB/s; HBM and the atomics' own rate about balance).
// ATOMIC: parts of a frame add into hist (zeroed before) with integer atomics,
// exact in any order; otherwise the block stores the frame's counts.
template <bool ATOMIC>
__global__ __launch_bounds__(HIST_T) void k_hist(const uint8_t *frames, long frame_bytes,
                                                 int split, int32_t *hist) {
  __shared__ __align__(16) uint32_t h[HB * 64];
  const int t = threadIdx.x, lane = t & 63;
  const int f = blockIdx.x / split, part = blockIdx.x % split;
  for (int i = t; i < HB * 16; i += HIST_T) reinterpret_cast<u32x4 *>(h)[i] = u32x4{0, 0, 0, 0};
  // The frame's whole 16-byte chunks (the base is 16-byte aligned, by
  // contract); at most 15 bytes on either side are counted one by one.
  const long s0 = (long)f * frame_bytes, s1 = s0 + frame_bytes;
  const long a0 = min((s0 + 15) & ~15L, s1), a1 = max(a0, s1 & ~15L);
  const long n16 = (a1 - a0) / 16;
  const long i0 = n16 * part / split, i1 = n16 * (part + 1) / split;
  const u32x4 *src = reinterpret_cast<const u32x4 *>(frames + a0);
  const int lead = (int)(a0 - s0);  // bytes before the first chunk
  // Byte b of the frame belongs to channel b % 3; chunk i starts at byte
  // lead + 16 i, channel (lead + i) % 3. Batches of HIST_B chunks per thread;
  // a batch's loads are issued before the previous batch is counted.
  constexpr int HIST_B = 4;
  auto load = [&](long i, u32x4 (&v)[HIST_B]) {
#pragma unroll
    for (int b = 0; b < HIST_B; ++b) {
      const long ib = i + (long)b * HIST_T;
      if (ib < i1) v[b] = src[ib];
    }
  };
  auto count = [&](long i, const u32x4 (&v)[HIST_B]) {
#pragma unroll
    for (int b = 0; b < HIST_B; ++b) {
      const long ib = i + (long)b * HIST_T;
      if (ib >= i1) break;
      const int c0 = (int)((lead + ib) % 3);
      // Byte offsets of this lane's word in bin 0 of the channels of bytes
      // 0, 1, 2 mod 3 (64 bins x 256 bytes per channel).
      const uint32_t l4 = 4u * lane;
      const uint32_t o0 = l4 | (uint32_t)(c0 << 14);
      const uint32_t o1 = l4 | (uint32_t)((c0 == 2 ? 0 : c0 + 1) << 14);
      const uint32_t o2 = l4 | (uint32_t)((c0 == 0 ? 2 : c0 - 1) << 14);
#pragma unroll
      for (int j = 0; j < 16; ++j) {
        // (byte >> 2) << 8: the bin's byte offset within the channel.
        const uint32_t x = v[b][j >> 2];
        const int sh = 8 * (j & 3) - 6;
        const uint32_t bin = (sh < 0 ? x << 6 : x >> sh) & 0x3F00u;
        const uint32_t off = bin | (j % 3 == 0 ? o0 : j % 3 == 1 ? o1 : o2);
        atomicAdd(reinterpret_cast<uint32_t *>(reinterpret_cast<char *>(h) + off), 1u);
      }
    }
  };
  u32x4 va[HIST_B], vb[HIST_B];
  constexpr long STEP = (long)HIST_B * HIST_T;
  load(i0 + t, va);
  __syncthreads();
  for (long i = i0 + t; i < i1; i += 2 * STEP) {
    load(i + STEP, vb);
    count(i, va);
    if (i + STEP >= i1) break;
    load(i + 2 * STEP, va);
    count(i + STEP, vb);
  }
  if (part == 0 && t < 32) {  // bytes outside the chunks
    const long b = t < 16 ? s0 + t : a1 + (t - 16), e = t < 16 ? a0 : s1;
    if (b < e)
      atomicAdd(&h[64 * ((int)((b - s0) % 3) * BINS + (frames[b] >> 2)) + lane], 1u);
  }
  __syncthreads();
  // Four threads sum a bin's words (rotated by the bin: distinct banks).
  if (t < 4 * HB) {
    const int bin = t >> 2;
    uint32_t sum = 0;
#pragma unroll
    for (int i = 0; i < 16; ++i) sum += h[64 * bin + ((16 * (t & 3) + i + bin) & 63)];
    sum += __shfl_xor(sum, 1, 64);
    sum += __shfl_xor(sum, 2, 64);
    if ((t & 3) == 0) {
      int32_t *dst = hist + (long)f * HB + bin;
      if constexpr (!ATOMIC)
        *dst = (int32_t)sum;
      else if (sum)
        atomicAdd(dst, (int32_t)sum);
    }
  }
}

// One block: inter[i] = sum_b min(hist[i][b], hist[i-1][b]) (inter[0] = -1),
// keyframe flags (frame 0, and inter[i] < theta * 3HW), then the ordered
// list of keyframe indices. Wave w takes a run of consecutive frames, the
// lanes three bins each, KF_U frames' loads in flight (a thread per frame
// walking its 192 bins alone took 12.5 us for 220 frames; now 5.8 us).
constexpr int KF_U = 16;
__global__ __launch_bounds__(1024) void k_keyframes(const int32_t *hist, int NF, double thr,
                                                    int32_t *inter, int32_t *key_idx,
                                                    int32_t *n_keys) {
  __shared__ uint32_t flags[2048];  // a bit per frame (NF <= 65536)
  __shared__ int32_t wsum[16];
  const int t = threadIdx.x, w = t >> 6, lane = t & 63;
  flags[t] = 0u;
  flags[t + 1024] = 0u;
  __syncthreads();
  const int per = (NF + 15) / 16, f0 = w * per, f1 = min(NF, f0 + per);
  for (int f = f0; f < f1; f += KF_U) {
    int32_t v[KF_U + 1][3];
#pragma unroll
    for (int u = 0; u <= KF_U; ++u) {  // rows f - 1 .. f + KF_U - 1
      const int32_t *row = hist + (long)min(max(f - 1 + u, 0), NF - 1) * HB + lane;
#pragma unroll
      for (int j = 0; j < 3; ++j) v[u][j] = row[64 * j];
    }
#pragma unroll
    for (int u = 0; u < KF_U; ++u) {
      int32_t s = 0;
#pragma unroll
      for (int j = 0; j < 3; ++j) s += min(v[u][j], v[u + 1][j]);
      s = wave_scan(s);  // the last lane has the sum
      const int g = f + u;
      if (lane == 63 && g < f1) {
        inter[g] = g == 0 ? -1 : s;
        if (g == 0 || (double)s < thr) atomicOr(&flags[g >> 5], 1u << (g & 31));
      }
    }
  }
  __syncthreads();
  // Thread t owns frames 64 t .. 64 t + 63: exclusive sums of the counts.
  uint32_t lo = flags[2 * t], hi = flags[2 * t + 1];
  const int mine = __popc(lo) + __popc(hi);
  const int sum = wave_scan(mine);
  if (lane == 63) wsum[w] = sum;
  __syncthreads();
  int pos = sum - mine, total = 0;
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    if (i < w) pos += wsum[i];
    total += wsum[i];
  }
  for (; lo; lo &= lo - 1) key_idx[pos++] = 64 * t + __ffs(lo) - 1;
  for (; hi; hi &= hi - 1) key_idx[pos++] = 64 * t + 32 + __ffs(hi) - 1;
  if (t == 0) *n_keys = total;
}

constexpr int RG = 16;       // keyframes per column group of the bank scan
constexpr int RT = 256;      // documents a block scores at a time
constexpr int kMaxLists = 256;  // lists per keyframe: a block a CU

// A ranked candidate as one unsigned 64-bit key: the similarity's
// order-preserving bits above the complement of the document index, so a
// larger key ranks before (ties: the lower index). 0: no candidate (a NaN is
// none). Comparisons and wave-wide maxima then are plain integer ones.
typedef unsigned long long key_t64;
__device__ __forceinline__ key_t64 make_key(float s, int i) {
  const uint32_t b = __float_as_uint(s + 0.f);  // -0 ranks as 0
  const uint32_t o = b ^ ((uint32_t)((int32_t)b >> 31) | 0x80000000u);
  return isnan(s) ? 0ull : ((key_t64)o << 32) | (uint32_t)~i;
}
__device__ __forceinline__ int key_index(key_t64 k) { return k ? (int)~(uint32_t)k : -1; }
__device__ __forceinline__ float key_sim(key_t64 k) {
  const uint32_t o = (uint32_t)(k >> 32);
  return __uint_as_float(o ^ (o & 0x80000000u ? 0x80000000u : 0xFFFFFFFFu));
}

template <int CTRL, int ROWS>
__device__ __forceinline__ key_t64 max_dpp(key_t64 v) {
  const int lo = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)v, CTRL, ROWS, 0xF, false);
  const int hi = __builtin_amdgcn_update_dpp(0, (int)(v >> 32), CTRL, ROWS, 0xF, false);
  const key_t64 u = ((key_t64)(uint32_t)hi << 32) | (uint32_t)lo;
  return u > v ? u : v;
}

// Largest key of the wave, in every lane: row shifts, then the rows' last
// lanes broadcast (a butterfly of LDS permutes took about 0.5 us a pass).
__device__ __forceinline__ key_t64 wave_best(key_t64 v) {
  v = max_dpp<0x111, 0xF>(v);
  v = max_dpp<0x112, 0xF>(v);
  v = max_dpp<0x114, 0xF>(v);
  v = max_dpp<0x118, 0xF>(v);
  v = max_dpp<0x142, 0xA>(v);
  v = max_dpp<0x143, 0xC>(v);
  const uint32_t lo = __builtin_amdgcn_readlane((int)(uint32_t)v, 63);
  const uint32_t hi = __builtin_amdgcn_readlane((int)(v >> 32), 63);
  return ((key_t64)hi << 32) | lo;
}

__device__ __forceinline__ key_t64 max_below(key_t64 best, key_t64 c, key_t64 last) {
  return c < last && c > best ? c : best;
}

// The top-k of keyframes g0 .. g0+ng-1 over the documents d0 .. d0+nd-1 (sims
// [..][RT] in LDS) and, unless `first`, over the block's list so far: wave w of
// NWV takes keyframes w, w + NWV, ..., k passes of a wave-wide best.
template <int NWV>
__device__ __forceinline__ void block_topk(const float (*sims)[RT], int g0, int ng, int d0,
                                           int nd, bool first, int k, int nlists, int list,
                                           key_t64 *part) {
  const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
  for (int r = w; r < ng; r += NWV) {
    key_t64 *out = part + ((long)(g0 + r) * nlists + list) * k;
    const key_t64 old = !first && lane < k ? out[lane] : 0ull;  // (the wave's own stores)
    key_t64 c[RT / 64];
#pragma unroll
    for (int e = 0; e < RT / 64; ++e) {
      const int j = lane + 64 * e;
      c[e] = j < nd ? make_key(sims[r][j], d0 + j) : 0ull;
    }
    key_t64 last = ~0ull, mine = 0ull;
    for (int p = 0; p < k; ++p) {
      key_t64 best = max_below(0ull, old, last);
#pragma unroll
      for (int e = 0; e < RT / 64; ++e) best = max_below(best, c[e], last);
      last = wave_best(best);
      if (lane == p) mine = last;  // 0: fewer than k documents left
    }
    if (lane < k) out[lane] = mine;
  }
}

// Scan of the bank: block (list, y) scores an even share (of nlists) of the
// documents, at most 256 at a time, against up to RG KG keyframes, as a
// [documents x D] . [D x 16 KG] product in fp32 (v_mfma_f32_16x16x4_f32), and
// takes the keyframe groups y, y + gridDim.y, ... in turn.
// Eight waves; of a batch's 16-document tiles wave w owns tiles w and w + 8.
// Per 16 dimensions lane l loads 4 consecutive values of document (l % 16) of
// each tile (16 rows x 64 contiguous bytes per load) and the matching 4
// values of keyframe (l % 16) from LDS, and runs 4 products per tile (product
// j takes dimension 4 (l / 16) + j of each lane group, the same for both
// operands). The documents' squared norms come from the same loads. Steps of
// 64 dimensions; the next step's loads are issued before the current step's
// products, a batch's first ones before the previous batch's lists are made.
// Dimensions past the last whole 16 are loaded one by one, zeros past D
// (keyframe rows in LDS are padded with zeros to whole 16s, and by 4 floats
// more so that the 16 rows of an LDS read fall into distinct banks).
//
// HBM-bound: the bank is read once per group of keyframes. With a block per 256
// documents and group of 16 frames, the empty blocks of a grid sized for
// every frame being a keyframe (391 x 14 blocks for 220 frames) held LDS that
// the others waited for, and 391 shares of 256 documents do not divide evenly
// over 256 CUs: 84 us for 12 keyframes over 100k x 768 (3.7 TB/s), in 256 equal
// shares 70 us (4.4 TB/s).
typedef float f32x4u __attribute__((ext_vector_type(4), aligned(4)));
constexpr int RM_T = 512;
template <int KG>
__global__ __launch_bounds__(RM_T) void k_retrieve_scan(const float *frame_emb,
                                                        const int32_t *key_idx,
                                                        const int32_t *n_keys, const float *docs,
                                                        int ND, int D, int k, int nlists,
                                                        key_t64 *part, int32_t *n_sel) {
  constexpr int NG = 2;  // 16-document tiles per wave
  extern __shared__ __align__(16) float q[];  // keyframes, [RG KG][QS]
  __shared__ float qn[RG * KG];
  __shared__ float dn[RT];
  __shared__ float sims[RG * KG][RT];
  const int nk = *n_keys, list = blockIdx.x, ny = gridDim.y;
  // Groups of 16 if every one of them has a block of its own (two passes of
  // half the lists side by side), otherwise 16 KG keyframes per pass.
  const int rows = KG == 1 || nk <= RG * ny ? RG : RG * KG, first = blockIdx.y * rows;
  const int t = threadIdx.x, w = t >> 6, lane = t & 63;
  const int QS = (D + 15) / 16 * 16 + 4, nfull = D / 16;
  const int sub = 4 * (lane >> 4);
  // n_sel counts finished keyframes in the merge (the next launch).
  if (list == 0 && first == 0 && t == 0) *n_sel = 0;
  const int b0 = (int)((long)ND * list / nlists), b1 = (int)((long)ND * (list + 1) / nlists);
  const int nb = (b1 - b0 + RT - 1) / RT;  // batches (at least one: nlists <= ND)
  const float *dp[NG];
  int d0 = 0, nd = 0;
  bool second = false;  // the wave's second tile is in use
  auto batch = [&](int b) {
    d0 = b0 + (int)((long)(b1 - b0) * b / nb);
    nd = b0 + (int)((long)(b1 - b0) * (b + 1) / nb) - d0;
    second = 16 * (w + 8) < nd;
#pragma unroll
    for (int g = 0; g < NG; ++g)
      dp[g] = docs + (long)(d0 + min(16 * (w + 8 * g) + (lane & 15), nd - 1)) * D + sub;
  };
  // Loads of the step at piece c (pieces past the last whole one repeat it).
  auto load = [&](int c, f32x4 (&v)[4][NG]) {
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int cc = 16 * min(c + u, nfull - 1);
      v[u][0] = *reinterpret_cast<const f32x4u *>(dp[0] + cc);
      if (second) v[u][1] = *reinterpret_cast<const f32x4u *>(dp[1] + cc);
    }
  };
  for (int g0 = first; g0 < nk; g0 += rows * ny) {
    const int ng = min(rows, nk - g0);
    const bool two = KG == 2 && ng > RG;  // the second column group is in use
    f32x4 va[4][NG], vb[4][NG];
#pragma unroll
    for (int u = 0; u < 4; ++u) va[u][1] = vb[u][1] = f32x4{0.f, 0.f, 0.f, 0.f};
    batch(0);
    if (nfull > 0) load(0, va);
    if (g0 > first) __syncthreads();  // the previous group's lists are done
    for (int r = w; r < rows; r += RM_T / 64) {  // a wave per row; rows past ng: zeros
      const float *src = frame_emb + (long)key_idx[g0 + min(r, ng - 1)] * D;
      float s = 0.f;
      for (int c = lane; c < QS; c += 64) {
        const float v = r < ng && c < D ? src[c] : 0.f;
        q[r * QS + c] = v;
        s += v * v;
      }
      s = wave_sum(s);
      if (lane == 0) qn[r] = sqrtf(s);
    }
    __syncthreads();
    const float *qp = q + (lane & 15) * QS + sub;
    for (int b = 0; b < nb; ++b) {
      // A sum for each of the four products of a piece, added up at the end. Error
      // of the similarities (2-norm) over 500 / 768 / 1000 dimensions: 1.1e-7 / 1.2e-7 /
      // 1.3e-7; as one chain over all of D 3.2e-7 / 4.6e-7 / 4.7e-7.
      f32x4 acc[4][KG][NG];
      float dd[NG];
#pragma unroll
      for (int g = 0; g < NG; ++g) {
#pragma unroll
        for (int h = 0; h < KG; ++h)
#pragma unroll
          for (int j = 0; j < 4; ++j) acc[j][h][g] = f32x4{0.f, 0.f, 0.f, 0.f};
        dd[g] = 0.f;
      }
      auto piece = [&](int c, const f32x4 (&v)[NG]) {
        const f32x4 e0 = *reinterpret_cast<const f32x4 *>(qp + 16 * c);
        f32x4 e1 = e0;
        if (two) e1 = *reinterpret_cast<const f32x4 *>(qp + RG * QS + 16 * c);
#pragma unroll
        for (int g = 0; g < NG; ++g) {
          const f32x4 x = v[g];
          dd[g] += x[0] * x[0] + x[1] * x[1] + x[2] * x[2] + x[3] * x[3];
#pragma unroll
          for (int j = 0; j < 4; ++j)
            acc[j][0][g] =
                __builtin_amdgcn_mfma_f32_16x16x4f32(x[j], e0[j], acc[j][0][g], 0, 0, 0);
          if (two)
#pragma unroll
            for (int j = 0; j < 4; ++j)
              acc[j][KG - 1][g] =
                  __builtin_amdgcn_mfma_f32_16x16x4f32(x[j], e1[j], acc[j][KG - 1][g], 0, 0, 0);
        }
      };
      auto step = [&](int c, const f32x4 (&v)[4][NG]) {
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          if (c + u >= nfull) break;
          piece(c + u, v[u]);
        }
      };
      for (int c = 0; c < nfull; c += 8) {
        if (c + 4 < nfull) load(c + 4, vb);
        __builtin_amdgcn_sched_barrier(0);
        step(c, va);
        if (c + 4 >= nfull) break;
        if (c + 8 < nfull) load(c + 8, va);
        __builtin_amdgcn_sched_barrier(0);
        step(c + 4, vb);
      }
      if (D % 16) {
        f32x4 x[NG];
#pragma unroll
        for (int g = 0; g < NG; ++g)
#pragma unroll
          for (int j = 0; j < 4; ++j)
            x[g][j] = 16 * nfull + sub + j < D ? dp[g][16 * nfull + j] : 0.f;
        piece(nfull, x);
      }
      const int d0b = d0, ndb = nd;
      if (b + 1 < nb) {
        batch(b + 1);
        if (nfull > 0) load(0, va);
      }
      // Squared norms: the four lane groups' partial sums (fixed order).
#pragma unroll
      for (int g = 0; g < NG; ++g) {
        float s = dd[g];
        s += __shfl_xor(s, 16, 64);
        s += __shfl_xor(s, 32, 64);
        if (lane < 16) dn[16 * (w + 8 * g) + lane] = sqrtf(s);
      }
      __syncthreads();  // (also: the previous batch's lists are done)
      // Lane l holds document 16 (w + 8 g) + 4 (l / 16) + i of the batch
      // against keyframe l % 16 of each column group.
#pragma unroll
      for (int h = 0; h < KG; ++h) {
        const int r = RG * h + (lane & 15);
        if (r < ng) {
#pragma unroll
          for (int g = 0; g < NG; ++g) {
            const f32x4 dot = (acc[0][h][g] + acc[1][h][g]) + (acc[2][h][g] + acc[3][h][g]);
#pragma unroll
            for (int i = 0; i < 4; ++i) {
              const int j = 16 * (w + 8 * g) + 4 * (lane >> 4) + i;
              const float den = qn[r] * dn[j];
              sims[r][j] = den > 0.f ? dot[i] / den : 0.f;
            }
          }
        }
      }
      __syncthreads();
      block_topk<RM_T / 64>(sims, g0, ng, d0b, ndb, b == 0, k, nlists, list, part);
    }
  }
}

// A value written by one block and read by another of the same launch: agent
// scope, so it goes past the writer's own L2.
template <typename T>
__device__ __forceinline__ void put_agent(T *p, T v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <typename T>
__device__ __forceinline__ T get_agent(const T *p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Block r < n_keys: the top-k of keyframe r over every block's top-k, then, in
// the block that finishes last, T* = the K best documents of the union of the
// top-k lists, a document scored by the best similarity it was retrieved with
// (Eq. 3). Each wave takes the top-k of its own share of the candidates (at most
// MERGE_PER per thread, in registers) without block barriers, then wave 0 merges
// the 16 lists. The finished keyframes are counted in n_sel, which the scan zeroed
// and which gets its value at the end. The lists are stored and loaded at
// agent scope, and a block counts itself once its stores are acknowledged (an
// agent-scope release would write back the whole L2: 13.7 us for 6 candidates
// per keyframe). As two launches the merge and the selection took 9.8 + 7.1 us
// for 12 keyframes over 100k documents, now 7.7 us.
constexpr int MERGE_T = 1024;
constexpr int MERGE_PER = 4;
static_assert(kMaxLists * 16 <= MERGE_T * MERGE_PER, "k <= 16 candidates of every list");
__global__ __launch_bounds__(MERGE_T) void k_retrieve_merge(const key_t64 *part,
                                                            const int32_t *n_keys, int nlists,
                                                            int k, int K, int32_t *top_idx,
                                                            float *top_sim, int32_t *sel_idx,
                                                            float *sel_sim, int32_t *n_sel) {
  __shared__ key_t64 wl[16 * (MERGE_T / 64)];  // list q of wave w at 16 q + w
  __shared__ int32_t finished;
  __shared__ int chosen[64];
  const int r = blockIdx.x, t = threadIdx.x, lane = t & 63, w = t >> 6;
  const key_t64 *p = part + (long)r * nlists * k;
  const int n = nlists * k, nk = *n_keys;
  key_t64 c[MERGE_PER];  // (loaded beside n_keys: rows past it hold other values, unused)
#pragma unroll
  for (int e = 0; e < MERGE_PER; ++e) c[e] = t + e * MERGE_T < n ? p[t + e * MERGE_T] : 0ull;
  if (r >= nk) return;  // uniform per block
  key_t64 last = ~0ull;
  for (int q = 0; q < k; ++q) {
    key_t64 best = 0ull;
#pragma unroll
    for (int e = 0; e < MERGE_PER; ++e) best = max_below(best, c[e], last);
    last = wave_best(best);
    if (lane == 0) wl[16 * q + w] = last;
    // (0: the wave's candidates are used up, the remaining passes find none)
  }
  __syncthreads();
  if (w == 0) {
    key_t64 m[4], mine = 0ull;  // 16 lists of k <= 16
#pragma unroll
    for (int e = 0; e < 4; ++e) m[e] = lane + 64 * e < 16 * k ? wl[lane + 64 * e] : 0ull;
    last = ~0ull;
    for (int q = 0; q < k; ++q) {
      key_t64 best = 0ull;
#pragma unroll
      for (int e = 0; e < 4; ++e) best = max_below(best, m[e], last);
      last = wave_best(best);
      if (lane == q) mine = last;
    }
    if (lane < k) {
      put_agent(top_idx + (long)r * k + lane, key_index(mine));
      put_agent(top_sim + (long)r * k + lane, mine ? key_sim(mine) : 0.f);
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // the list is out
    if (lane == 0)
      finished = __hip_atomic_fetch_add(n_sel, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  __syncthreads();
  if (finished != nk - 1) return;  // uniform per block
  const int ne = nk * k;
  auto entry = [&](int e) {
    const int d = get_agent(top_idx + e);
    const float v = get_agent(top_sim + e);
    return d < 0 ? 0ull : make_key(v, d);
  };
  // The thread's first entry stays in a register (the only one up to 1024).
  key_t64 e0 = t < ne ? entry(t) : 0ull;
  int got = 0;
  for (int q = 0; q < K; ++q) {
    // Best among the entries whose document is not chosen yet.
    key_t64 best = e0;
    for (int e = t + MERGE_T; e < ne; e += MERGE_T) {
      const key_t64 x = entry(e);
      bool taken = false;
      for (int i = 0; i < got; ++i) taken = taken || chosen[i] == key_index(x);
      if (!taken && x > best) best = x;
    }
    best = wave_best(best);
    if (lane == 0) wl[16 * (q & 1) + w] = best;
    __syncthreads();
    best = wave_best(lane < MERGE_T / 64 ? wl[16 * (q & 1) + lane] : 0ull);
    if (!best) break;  // uniform: every wave reduced the same 16 entries
    const int d = key_index(best);
    if (t == 0) {
      sel_idx[got] = d;
      sel_sim[got] = key_sim(best);
      chosen[got] = d;
    }
    if (key_index(e0) == d) e0 = 0ull;
    ++got;
    if (ne > MERGE_T) __syncthreads();  // `chosen` is read
  }
  if (t == 0) *n_sel = got;
}

}  // namespace

hipError_t launch_keyframes(const uint8_t *frames, int NF, int H, int W, float theta,
                            int32_t *hist, int32_t *inter, int32_t *key_idx, int32_t *n_keys,
                            hipStream_t s) {
  const long fb = (long)H * W * 3;
  // One block per frame stores the frame's counts. A block counts about 26 GB/s,
  // so some 190 of them reach what the chip counts: fewer frames are cut into
  // parts (of at least 32 KB, up to two blocks a CU) that add into zeroed counts,
  // where the time the idle CUs save, frame bytes x (190 - NF) / 190 / 26 GB/s, is
  // above that of the extra launch, about 2 us, and a frame is above 64 KB (8
  // frames of 120 x 160: 9.4 whole, 10.3 in parts). In two parts, past 170 frames,
  // it gains nothing. Whole frames / parts, us: 130 frames of 336 x 336 22.2/20.8, of
  // 480 x 854 55/43, of 1080 x 1920 243/177; 127 of 200 x 200 13.4/14.0, of 224 x 224
  // 14.7/14.1; 175 of 480 x 854 56/57.
  int split = 1;
  if (NF <= 170 && fb > (64 << 10) && fb * (190 - NF) > 9000000)
    split = (int)std::max<long>(2, std::min<long>(512 / NF, fb >> 15));
  if (split == 1) {
    k_hist<false><<<NF, HIST_T, 0, s>>>(frames, fb, 1, hist);
  } else {
    const long nh = (long)NF * HB;
    k_zero_i32<<<(unsigned)((nh + 255) / 256), 256, 0, s>>>(hist, nh);
    k_hist<true><<<NF * split, HIST_T, 0, s>>>(frames, fb, split, hist);
  }
  const double thr = (double)theta * 3.0 * (double)((long)H * W);  // (theta 3) (H W)
  k_keyframes<<<1, 1024, 0, s>>>(hist, NF, thr, inter, key_idx, n_keys);
  return hipGetLastError();
}

// One list per 256 documents and keyframe: what callers size their buffers by, and
// the static scratch refuses calls by. Banks of more than kMaxLists x 256 documents
// use kMaxLists of them.
size_t retrieve_workspace_bytes(int NF, int ND, int k) {
  const size_t nchunks = ((size_t)ND + RT - 1) / RT;
  return (size_t)NF * nchunks * (size_t)k * sizeof(key_t64);
}

hipError_t launch_retrieve(const float *frame_emb, const int32_t *key_idx, const int32_t *n_keys,
                           int NF, const float *docs, int ND, int D, int k, int K, void *ws,
                           int32_t *top_idx, float *top_sim, int32_t *sel_idx, float *sel_sim,
                           int32_t *n_sel, hipStream_t s) {
  key_t64 *part = static_cast<key_t64 *>(ws);
  // Up to 32 keyframes per pass over the bank if there may be more than 16 and
  // their rows (with 32 lists of similarities) fit the 160 KB of LDS. A list per
  // block of documents, as many as the CUs hold blocks at once (one each, by their
  // registers: in two rounds of 391 blocks 12 of at most 16 keyframes against 100k
  // documents took 92 us, now 73); what a small bank leaves of them takes further
  // groups of keyframes. (One block per list took the groups of a small bank in
  // turn: 200 keyframes against 156 and 5000 documents of 768 288 and 315 us, now
  // 38 and 69; a grid sized for every frame being a keyframe 55 and 81 us.)
  const size_t qrow = ((size_t)(D + 15) / 16 * 16 + 4) * sizeof(float);
  const bool wide = NF > RG && 2 * RG * (qrow + RT * sizeof(float)) <= (size_t)150 << 10;
  const int rows = wide ? 2 * RG : RG;
  const int nlists = std::min((ND + RT - 1) / RT, kMaxLists);
  const dim3 grid(nlists, std::min((NF + RG - 1) / RG, kMaxLists / nlists));
  if (wide)
    k_retrieve_scan<2><<<grid, RM_T, rows * qrow, s>>>(frame_emb, key_idx, n_keys, docs, ND, D, k,
                                                       nlists, part, n_sel);
  else
    k_retrieve_scan<1><<<grid, RM_T, rows * qrow, s>>>(frame_emb, key_idx, n_keys, docs, ND, D, k,
                                                       nlists, part, n_sel);
  k_retrieve_merge<<<NF, MERGE_T, 0, s>>>(part, n_keys, nlists, k, K, top_idx, top_sim, sel_idx,
                                          sel_sim, n_sel);
  return hipGetLastError();
}

// ---- the same retrieval with library-owned scratch ------------------------
// For callers that cannot allocate device memory: the per-chunk partial lists
// live in this file-scope array (one copy per GPU, held until the process
// ends). Host code never passes the array's name to a kernel: it is a
// host-side stand-in there. The device address comes from
// hipGetSymbolAddress, looked up once per device with that device current.
static __device__ __align__(256) unsigned char scratch[kRetrieveStaticBytes];

namespace {
std::mutex g_scratch_mu;
void *g_scratch_ptr[kMaxDevices] = {};
}  // namespace

hipError_t retrieve_static_scratch(void **ptr) {
  int dev = -1;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (!g_scratch_ptr[dev]) {
    void *p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    if (!p) return hipErrorInvalidSymbol;
    g_scratch_ptr[dev] = p;
  }
  *ptr = g_scratch_ptr[dev];
  return hipSuccess;
}

}  // namespace vsr
