// Random-forest feasibility model (Sec. 4.2, hidden constraints): a classification
// forest fitted to the feasible / infeasible labels of the observations predicts the
// probability of feasibility that multiplies the expected improvement.
//
// Trees are CART trees with Gini impurity grown on bootstrap samples with a random
// feature subset per node; all random choices come from Philox4x64-10 streams (key
// (seed, 0), counter (tree, stream, block, 3); stream 0 the bootstrap, stream k + 1
// the feature subset of node k), so the trees are a deterministic function of the
// inputs. Split qualities Q = pos_L neg_L / c_L + pos_R neg_R / c_R (the Gini impurity
// of the children weighted by their sizes, halved) are compared exactly as fractions
// of 64-bit integers: the smallest Q wins, then the smallest feature, then the
// smallest threshold; a split is taken only if Q is below the node's own
// pos neg / c. A threshold is the largest value sent left.
//
// Training: features are replaced by their ranks among the observations' distinct values
// (one workgroup per feature), then one workgroup per tree grows it level by level: the
// nodes of a level are independent, one wavefront takes one at a time, and the children
// are numbered by a prefix sum over the level, which is breadth-first order. A node of at
// most 64 samples keeps one sample per lane and counts, for each, the samples of smaller
// or equal rank; a larger one counts samples per rank in LDS and scans the counts. Every
// boundary between distinct values is scored, the best of all tried features reduced over
// the wavefront, and the node's sample range partitioned stably.
// Prediction: a configuration's features become ranks too (x <= threshold exactly when
// fewer distinct values lie below x than up to the threshold), so a node is 8 bytes and a
// workgroup keeps many trees and its configurations' ranks in LDS; a lane walks two trees
// at a time. 1,048,576 configurations and 64 trees take 389 us, bound by the random LDS
// reads of the walks; 16-byte nodes read from the caches took 1,060 us, bound by one
// address per lane and cycle. Few trees are still walked that way (forest_direct below).
#include <algorithm>

#include "common.h"

namespace bgp {
namespace {

__device__ __forceinline__ void philox4x64(uint64_t c0, uint64_t c1, uint64_t c2, uint64_t c3,
                                           uint64_t k0, uint64_t k1, uint64_t out[4]) {
  constexpr uint64_t M0 = 0xD2E7470EE14C6C93ull, M1 = 0xCA5A826395121157ull;
  constexpr uint64_t W0 = 0x9E3779B97F4A7C15ull, W1 = 0xBB67AE8584CAA73Bull;
#pragma unroll
  for (int r = 0; r < 10; ++r) {
    if (r) {
      k0 += W0;
      k1 += W1;
    }
    const uint64_t hi0 = __umul64hi(M0, c0), lo0 = M0 * c0;
    const uint64_t hi1 = __umul64hi(M1, c2), lo1 = M1 * c2;
    const uint64_t n0 = hi1 ^ c1 ^ k0, n2 = hi0 ^ c3 ^ k1;
    c0 = n0;
    c1 = lo1;
    c2 = n2;
    c3 = lo0;
  }
  out[0] = c0;
  out[1] = c1;
  out[2] = c2;
  out[3] = c3;
}

// word q of stream (t, s)
__device__ __forceinline__ uint64_t stream_word(uint64_t seed, int t, int s, int q) {
  uint64_t w[4];
  philox4x64((uint64_t)t, (uint64_t)s, (uint64_t)(q >> 2), 3, seed, 0, w);
  const int r = q & 3;
  return r == 0 ? w[0] : (r == 1 ? w[1] : (r == 2 ? w[2] : w[3]));
}

template <typename T>
__device__ __forceinline__ void stage(T &dst, const T &src) {
  static_assert(sizeof(T) % 4 == 0, "word copy");
  const uint32_t *s = reinterpret_cast<const uint32_t *>(&src);
  uint32_t *d = reinterpret_cast<uint32_t *>(&dst);
  for (int q = threadIdx.x; q < (int)(sizeof(T) / 4); q += blockDim.x) d[q] = s[q];
}

// a/b < c/d for nonnegative fractions with a, c < 2^40 and b, d < 2^24
__device__ __forceinline__ bool frac_less(uint64_t a, uint64_t b, uint64_t c, uint64_t d) {
  return a * d < c * b;
}

__device__ __forceinline__ double feature_of(const ForestDesc &D, const CotCols &cols, int p, int q,
                                             int64_t j) {
  const int kind = D.kind[p];
  if (kind == GP_REAL) return static_cast<const double *>(cols.col[p])[j];
  if (kind == GP_PERM) return (double)static_cast<const int32_t *>(cols.col[p])[j * D.m[p] + q];
  return (double)static_cast<const int32_t *>(cols.col[p])[j];
}

__global__ __launch_bounds__(256) void forest_features_k(const ForestDesc *dd, const CotCols cols0,
                                                          int64_t count, int64_t ld, double *X) {
  __shared__ ForestDesc D;
  __shared__ CotCols cols;
  stage(D, *dd);
  stage(cols, cols0);
  __syncthreads();
  const int64_t j = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (j >= count) return;
  for (int p = 0; p < D.d; ++p)
    for (int q = 0; q < D.m[p]; ++q) X[(int64_t)(D.fofs[p] + q) * ld + j] = feature_of(D, cols, p, q, j);
}

// Ranks of feature f (workgroup f): rank[f][i] = distinct values below x_i, val[f][r] = the
// distinct value of rank r, nd[f] their number. Every observation is compared with the
// first occurrence of each value; n^2 comparisons per feature, all features at once.
constexpr int kRankThreads = 1024;
__global__ __launch_bounds__(kRankThreads) void forest_ranks_k(const double *X, int32_t n,
                                                               uint16_t *rank, double *val,
                                                               int32_t *nd) {
  __shared__ double x[kMaxN];
  __shared__ uint8_t first[kMaxN];
  __shared__ int cnt;
  const int f = blockIdx.x, tid = threadIdx.x;
  if (tid == 0) cnt = 0;
  for (int i = tid; i < n; i += kRankThreads) x[i] = X[(int64_t)f * n + i];
  __syncthreads();
  for (int i = tid; i < n; i += kRankThreads) {
    const double v = x[i];
    int seen = 0;  // (no early exit: the unrolled loads are in flight together)
#pragma unroll 16
    for (int j = 0; j < i; ++j) seen |= x[j] == v ? 1 : 0;
    first[i] = seen ? 0 : 1;
    if (!seen) atomicAdd(&cnt, 1);
  }
  __syncthreads();
  for (int i = tid; i < n; i += kRankThreads) {
    const double v = x[i];
    int r = 0;
#pragma unroll 16
    for (int j = 0; j < n; ++j) r += (first[j] && x[j] < v) ? 1 : 0;
    rank[(int64_t)f * n + i] = (uint16_t)r;
    if (first[i]) val[(int64_t)f * n + r] = v;
  }
  if (tid == 0) nd[f] = cnt;
}

// A split candidate: its quality num / den, and the tried feature's place and the rank as
// one tie-breaking key (0xffffffff: none)
struct Split {
  uint64_t num;
  uint32_t den, key, left;  // left: samples sent left
};
__device__ __forceinline__ bool split_before(const Split &a, const Split &b) {
  if (a.key == 0xffffffffu || b.key == 0xffffffffu) return a.key < b.key;
  const uint64_t l = a.num * b.den, r = b.num * a.den;
  return l < r || (l == r && a.key < b.key);
}
// The split after which cl samples (pl of them feasible) of the node's c (pos) lie left.
__device__ __forceinline__ Split split_of(uint32_t cl, uint32_t pl, uint32_t c, uint32_t pos,
                                          uint32_t key) {
  const uint64_t cr = c - cl, pr = pos - pl;
  Split s;
  s.num = (uint64_t)pl * (cl - pl) * cr + pr * (cr - pr) * cl;
  s.den = (uint32_t)(cl * cr);
  s.key = key;
  s.left = cl;
  return s;
}

__device__ __forceinline__ uint64_t shfl_xor_u64(uint64_t v, int o) {
  const uint32_t lo = (uint32_t)__shfl_xor((int)(uint32_t)v, o);
  const uint32_t hi = (uint32_t)__shfl_xor((int)(uint32_t)(v >> 32), o);
  return (uint64_t)lo | ((uint64_t)hi << 32);
}

// Orders a wavefront's own LDS accesses (its LDS instructions are performed in order; this
// keeps the compiler from moving them).
__device__ __forceinline__ void wave_order() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// A packed node for prediction: an internal node has the top bit set, its feature above its
// threshold's rank and its left child; a leaf is its value (a nonnegative double).
__device__ __forceinline__ uint64_t pack_split(int f, uint32_t rank, uint32_t left) {
  return 0x8000000000000000ull | ((uint64_t)(uint32_t)f << 32) | (rank << 16) | left;
}

// Samples are 16-bit words: the observation's index and its label in the top bit.
constexpr uint32_t kLabelBit = 0x8000u;
static_assert(kMaxN <= 0x8000, "an index and a label in 16 bits");
__global__ __launch_bounds__(1024) void forest_train_k(const ForestDesc *dd, const uint16_t *rank,
                                                        const double *val, const int32_t *nd,
                                                        const uint8_t *y, ForestNode *nodes_all,
                                                        uint64_t *pack_all, int32_t *aux_all,
                                                        int32_t *n_nodes_out, int32_t bins_wave) {
  extern __shared__ uint32_t lds[];  // [waves][bins_wave] counts, then two sample orders
  __shared__ int wsum[16];
  typedef __attribute__((address_space(4))) const ForestDesc cdesc;
  const cdesc &D = *(const cdesc *)dd;
  const int t = blockIdx.x, tid = threadIdx.x, lane = tid & 63;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6), nw = blockDim.x >> 6;
  const int n = D.n, F = D.F, mtry = D.mtry;
  uint32_t *bins = lds + wv * bins_wave;
  uint16_t *idx = reinterpret_cast<uint16_t *>(lds + nw * bins_wave), *nxt = idx + n;
  ForestNode *nodes = nodes_all + (int64_t)t * D.cap;
  uint64_t *pack = pack_all + (int64_t)t * D.cap;
  int32_t *aux = aux_all + (int64_t)t * D.cap * 3;  // start, end, samples sent left (0: leaf)
  // bootstrap sample: index i from word i of stream (t, 0)
  for (int i = tid; i < n; i += blockDim.x) {
    const uint32_t o = (uint32_t)__umul64hi(stream_word(D.seed, t, 0, i), (uint64_t)n);
    idx[i] = (uint16_t)(o | (y[o] != 0 ? kLabelBit : 0u));
  }
  if (tid == 0) {
    aux[0] = 0;
    aux[1] = n;
  }
  __syncthreads();
  int k0 = 0, k1 = 1, s_nn = 1;
  for (int depth = 0; k0 < k1; ++depth) {
    for (int k = k0 + wv; k < k1; k += nw) {  // one node per wavefront
      const int start = __builtin_amdgcn_readfirstlane(aux[3 * k]);
      const int c = __builtin_amdgcn_readfirstlane(aux[3 * k + 1]) - start;
      int pos = 0;
      for (int i0 = 0; i0 < c; i0 += 64) {
        const bool p = i0 + lane < c && (idx[start + i0 + lane] & kLabelBit);
        pos += __popcll(__ballot(p));
      }
      const double leaf_val = (double)pos / (double)c;
      const bool leaf = pos == 0 || pos == c || c < D.min_split || depth >= D.max_depth;
      Split best{0, 1, 0xffffffffu, 0};
      int feat = 0;  // lane q: the q-th smallest of the features tried at this node
      if (!leaf) {
        // partial Fisher-Yates over 0..F-1: lane q follows position q's pick back through
        // the swaps before it
        int r = lane;
        if (lane < mtry)
          r = lane + (int)__umul64hi(stream_word(D.seed, t, k + 1, lane), (uint64_t)(F - lane));
        int pick = r;
        for (int p = mtry - 1; p >= 0; --p) {
          const int rp = __builtin_amdgcn_readlane(r, p);
          if (p < lane) pick = pick == p ? rp : (pick == rp ? p : pick);
        }
        int place = 0;
        for (int q = 0; q < mtry; ++q) place += __builtin_amdgcn_readlane(pick, q) < pick ? 1 : 0;
        for (int q = 0; q < mtry; ++q) {
          const int pl = __builtin_amdgcn_readlane(place, q), v = __builtin_amdgcn_readlane(pick, q);
          feat = lane == pl ? v : feat;
        }
        if (c <= 64) {
          const uint32_t s = lane < c ? idx[start + lane] : 0u;
          for (int q0 = 0; q0 < mtry; q0 += 4) {
            uint32_t rk[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {  // four features' loads in flight
              const int f = __builtin_amdgcn_readlane(feat, min(q0 + u, mtry - 1));
              rk[u] = lane < c ? rank[(int64_t)f * n + (s & (kLabelBit - 1))] : 0xffffu;
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) {
              if (q0 + u >= mtry) break;
              const uint32_t w = (rk[u] << 1) | (s >> 15);
              uint32_t acc = 0;  // samples of rank <= this lane's: count | feasible << 16
              for (int i = 0; i < c; ++i) {
                const uint32_t o = (uint32_t)__builtin_amdgcn_readlane((int)w, i);
                acc += (o >> 1) <= rk[u] ? (1u | ((o & 1u) << 16)) : 0u;
              }
              const uint32_t cl = acc & 0xffffu;
              if (lane < c && cl < (uint32_t)c) {
                const Split sp = split_of(cl, acc >> 16, c, pos, ((uint32_t)(q0 + u) << 16) | rk[u]);
                if (split_before(sp, best)) best = sp;
              }
            }
          }
        } else {
          for (int q = 0; q < mtry; ++q) {
            const int f = __builtin_amdgcn_readlane(feat, q);
            const int nv = __builtin_amdgcn_readfirstlane(nd[f]);
            const int per = ((nv + 63) >> 6) | 1;  // ranks per lane, odd: no bank conflicts
            wave_order();
            for (int i = lane; i < per * 64; i += 64) bins[i] = 0u;
            wave_order();
            const uint16_t *rf = rank + (int64_t)f * n;
            for (int i = lane; i < c; i += 64) {
              const uint32_t s = idx[start + i];
              atomicAdd(&bins[rf[s & (kLabelBit - 1)]], 1u | ((s >> 15) << 16));
            }
            wave_order();
            uint32_t sum = 0;
            for (int i = 0; i < per; ++i) sum += bins[lane * per + i];
            uint32_t run = sum;  // inclusive scan over the lanes
#pragma unroll
            for (int o = 1; o < 64; o <<= 1) {
              const uint32_t v = (uint32_t)__shfl_up((int)run, o);
              run += lane >= o ? v : 0u;
            }
            run -= sum;
            for (int i = 0; i < per; ++i) {
              const uint32_t b = bins[lane * per + i];
              run += b;
              const uint32_t cl = run & 0xffffu;
              if (b != 0u && cl < (uint32_t)c) {
                const Split sp = split_of(cl, run >> 16, c, pos, ((uint32_t)q << 16) | (uint32_t)(lane * per + i));
                if (split_before(sp, best)) best = sp;
              }
            }
          }
        }
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) {
          Split s2;
          s2.num = shfl_xor_u64(best.num, o);
          s2.den = (uint32_t)__shfl_xor((int)best.den, o);
          s2.key = (uint32_t)__shfl_xor((int)best.key, o);
          s2.left = (uint32_t)__shfl_xor((int)best.left, o);
          if (split_before(s2, best)) best = s2;
        }
      }
      // a split only on a strict improvement over the node's own pos neg / c
      const bool take = best.key != 0xffffffffu &&
                        frac_less(best.num, best.den, (uint64_t)pos * (uint64_t)(c - pos), (uint64_t)c);
      const int q = (int)(best.key >> 16);
      const uint32_t rb = best.key & 0xffffu;
      const int f = __builtin_amdgcn_readlane(feat, __builtin_amdgcn_readfirstlane(take ? q : 0));
      if (lane == 0) {
        nodes[k].feature = take ? f : -1;
        nodes[k].left = -1;
        nodes[k].val = take ? val[(int64_t)f * n + rb] : leaf_val;
        pack[k] = take ? pack_split(f, rb, 0) : __builtin_bit_cast(uint64_t, leaf_val);
        aux[3 * k + 2] = take ? (int)best.left : 0;
      }
      if (take) {  // stable partition: ranks up to the threshold's first
        const uint16_t *rf = rank + (int64_t)f * n;
        int nl = start, nr = start + (int)best.left;
        for (int i0 = 0; i0 < c; i0 += 64) {
          const bool in = i0 + lane < c;
          const uint32_t s = in ? idx[start + i0 + lane] : 0u;
          const bool l = in && rf[s & (kLabelBit - 1)] <= rb;
          const uint64_t bl = __ballot(l), br = __ballot(in && !l), below = (1ull << lane) - 1ull;
          if (in) nxt[l ? nl + __popcll(bl & below) : nr + __popcll(br & below)] = (uint16_t)s;
          nl += __popcll(bl);
          nr += __popcll(br);
        }
      }
    }
    __syncthreads();
    // number the children in node order
    const int lvl0 = k0, lvl1 = k1;
    for (int b0 = lvl0; b0 < lvl1; b0 += blockDim.x) {
      const int k = b0 + tid;
      const int sent = k < lvl1 ? aux[3 * k + 2] : 0;
      const uint64_t bal = __ballot(sent > 0);
      if (lane == 0) wsum[wv] = __popcll(bal);
      __syncthreads();
      int before = 0, total = 0;
      for (int w = 0; w < nw; ++w) {
        before += w < wv ? wsum[w] : 0;
        total += wsum[w];
      }
      if (sent > 0) {
        const int l = s_nn + 2 * (before + __popcll(bal & ((1ull << lane) - 1ull)));
        const int start = aux[3 * k], end = aux[3 * k + 1];
        nodes[k].left = l;
        pack[k] |= (uint64_t)(uint32_t)l;
        aux[3 * l] = start;
        aux[3 * l + 1] = start + sent;
        aux[3 * (l + 1)] = start + sent;
        aux[3 * (l + 1) + 1] = end;
      }
      s_nn += 2 * total;
      __syncthreads();
    }
    k0 = lvl1;
    k1 = s_nn;
    uint16_t *const sw = idx;
    idx = nxt;
    nxt = sw;
  }
  if (tid == 0) n_nodes_out[t] = s_nn;
}

// The outputs of configuration j: the mean of its leaves and the acquisition value.
__device__ __forceinline__ void forest_store(double sum, int n_trees, int64_t j, const float *ei,
                                             const uint8_t *mask, float eps_f, float *p_out,
                                             float *acq) {
  const float pf = (float)(sum / (double)n_trees);
  p_out[j] = pf;
  if (acq) {
    const bool allowed = !mask || mask[j];
    acq[j] = (allowed && pf > eps_f) ? ei[j] * pf : 0.0f;
  }
}

// Prediction. lofs[t]: tree t's first node in its batch's LDS; bstart[0..nbatch]: first tree
// of each batch (of trees that fit tree_words 8-byte nodes together).
__global__ __launch_bounds__(1024) void forest_predict_k(
    const ForestDesc *dd, const uint64_t *pack, const int32_t *n_nodes, const int32_t *lofs,
    const int32_t *bstart, int nbatch, int tree_words, const double *val, const int32_t *nd,
    const CotCols cols0, int64_t M, const float *ei, const uint8_t *mask, float eps_f,
    float *p_out, float *acq) {
  extern __shared__ uint64_t trees[];  // [tree_words], then ranks [waves][F][64]
  typedef __attribute__((address_space(4))) const ForestDesc cdesc;
  typedef __attribute__((address_space(1))) const int32_t gint;
  typedef __attribute__((address_space(1))) const double gdbl;
  const cdesc &D = *(const cdesc *)dd;
  const int tid = threadIdx.x, lane = tid & 63, T = blockDim.x;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  uint16_t *rk = reinterpret_cast<uint16_t *>(trees + tree_words) + (int64_t)wv * D.F * 64;
  bool loaded = false;  // one batch stays in LDS for every configuration
  for (int64_t j0 = (int64_t)blockIdx.x * T; j0 < M; j0 += (int64_t)gridDim.x * T) {
    const int64_t j = min(j0 + tid, M - 1);
    // ranks of the configuration's features: the distinct values below each
    for (int p = 0; p < D.d; ++p) {
      for (int q = 0; q < D.m[p]; ++q) {
        double x;
        if (D.kind[p] == GP_REAL) x = ((const gdbl *)cols0.col[p])[j];
        else if (D.kind[p] == GP_PERM) x = (double)((const gint *)cols0.col[p])[j * D.m[p] + q];
        else x = (double)((const gint *)cols0.col[p])[j];
        const int f = D.fofs[p] + q;
        const double *vf = val + (int64_t)f * D.n;
        int lo = 0, len = nd[f];
        while (len > 0) {
          const int h = len >> 1;
          const bool less = vf[lo + h] < x;
          lo = less ? lo + h + 1 : lo;
          len = less ? len - h - 1 : h;
        }
        rk[f * 64 + lane] = x != x ? (uint16_t)0xffffu : (uint16_t)lo;  // a NaN goes right
      }
    }
    double acc = 0.0;
    for (int b = 0; b < nbatch; ++b) {
      const int t0 = bstart[b], t1 = bstart[b + 1];
      if (!loaded) {
        __syncthreads();  // the batch before is no longer read
        for (int t = t0 + wv; t < t1; t += T >> 6) {
          const uint64_t *src = pack + (int64_t)t * D.cap;
          const int nn = n_nodes[t], o = lofs[t];
          for (int i = lane; i < nn; i += 64) trees[o + i] = src[i];
        }
        __syncthreads();
        loaded = nbatch == 1;
      }
      int t = t0;
      for (; t + 2 <= t1; t += 2) {  // two walks at a time, their leaves added in tree order
        const uint64_t *ta = trees + lofs[t], *tb = trees + lofs[t + 1];
        uint64_t a = ta[0], c = tb[0];
        while ((int64_t)a < 0 || (int64_t)c < 0) {
          const bool ia = (int64_t)a < 0, ic = (int64_t)c < 0;
          const uint32_t la = (uint32_t)a, lc = (uint32_t)c;
          const uint32_t fa = ia ? (uint32_t)(a >> 32) & 0xffffu : 0u, fc = ic ? (uint32_t)(c >> 32) & 0xffffu : 0u;
          const uint32_t ra = rk[fa * 64 + lane], rc = rk[fc * 64 + lane];
          const uint32_t na = ia ? (la & 0xffffu) + (ra > (la >> 16) ? 1u : 0u) : 0u;
          const uint32_t nc = ic ? (lc & 0xffffu) + (rc > (lc >> 16) ? 1u : 0u) : 0u;
          const uint64_t a2 = ta[na], c2 = tb[nc];
          a = ia ? a2 : a;
          c = ic ? c2 : c;
        }
        acc += __builtin_bit_cast(double, a);
        acc += __builtin_bit_cast(double, c);
      }
      for (; t < t1; ++t) {
        const uint64_t *ta = trees + lofs[t];
        uint64_t a = ta[0];
        while ((int64_t)a < 0) {
          const uint32_t la = (uint32_t)a;
          const uint32_t ra = rk[((uint32_t)(a >> 32) & 0xffffu) * 64 + lane];
          a = ta[(la & 0xffffu) + (ra > (la >> 16) ? 1u : 0u)];
        }
        acc += __builtin_bit_cast(double, a);
      }
    }
    if (j0 + tid < M) forest_store(acc, D.n_trees, j, ei, mask, eps_f, p_out, acq);
  }
}

// Prediction by few trees: a wavefront per 64 configurations, their features' own values in
// LDS and 16-byte nodes read through the caches, two walks at a time. It has neither the
// binary search per feature nor the copy of the trees to LDS.
__global__ __launch_bounds__(64) void forest_predict_direct_k(
    const ForestDesc *dd, const ForestNode *nodes, const CotCols cols0, int64_t M, const float *ei,
    const uint8_t *mask, float eps_f, float *p_out, float *acq) {
  extern __shared__ double feat[];  // [F][64]
  __shared__ ForestDesc D;
  __shared__ CotCols cols;
  stage(D, *dd);
  stage(cols, cols0);
  __syncthreads();
  const int lane = threadIdx.x;
  const int64_t j = (int64_t)blockIdx.x * 64 + lane;
  if (j >= M) return;
  for (int p = 0; p < D.d; ++p)
    for (int q = 0; q < D.m[p]; ++q) feat[(D.fofs[p] + q) * 64 + lane] = feature_of(D, cols, p, q, j);
  // (a NaN compares false and goes right)
  auto child = [&](const ForestNode &a) {
    return a.left + (feat[a.feature * 64 + lane] <= a.val ? 0 : 1);
  };
  double acc = 0.0;
  int t = 0;
  for (; t + 2 <= D.n_trees; t += 2) {  // their leaves are added in tree order
    const ForestNode *na = nodes + (int64_t)t * D.cap, *nb = na + D.cap;
    ForestNode a = na[0], b = nb[0];
    while (a.feature >= 0 || b.feature >= 0) {
      const ForestNode a2 = na[a.feature >= 0 ? child(a) : 0], b2 = nb[b.feature >= 0 ? child(b) : 0];
      if (a.feature >= 0) a = a2;
      if (b.feature >= 0) b = b2;
    }
    acc += a.val;
    acc += b.val;
  }
  if (t < D.n_trees) {
    const ForestNode *nt = nodes + (int64_t)t * D.cap;
    ForestNode a = nt[0];
    while (a.feature >= 0) a = nt[child(a)];
    acc += a.val;
  }
  forest_store(acc, D.n_trees, j, ei, mask, eps_f, p_out, acq);
}

}  // namespace

hipError_t launch_forest_features(const ForestDesc *dd, const CotCols &cols, int64_t count,
                                  int64_t ld, double *X, hipStream_t s) {
  if (count <= 0) return hipSuccess;
  hipLaunchKernelGGL(forest_features_k, dim3((unsigned)((count + 255) / 256)), dim3(256), 0, s, dd,
                     cols, count, ld, X);
  return hipGetLastError();
}

hipError_t launch_forest_ranks(const double *X, int32_t n, int32_t F, uint16_t *rank, double *val,
                               int32_t *nd, hipStream_t s) {
  if (n < 1 || n > kMaxN || F < 1) return hipErrorInvalidValue;
  hipLaunchKernelGGL(forest_ranks_k, dim3((unsigned)F), dim3(kRankThreads), 0, s, X, n, rank, val, nd);
  return hipGetLastError();
}

hipError_t launch_forest_train(const ForestDesc *dd, const ForestDesc &hd, const uint16_t *rank,
                               const double *val, const int32_t *nd, const uint8_t *y,
                               ForestNode *nodes, uint64_t *pack, int32_t *aux, int32_t *n_nodes,
                               hipStream_t s) {
  if (hd.n_trees <= 0) return hipSuccess;
  // a wavefront's counts cover n distinct values; as many wavefronts as the LDS holds
  const int bins = 64 * (((hd.n + 63) / 64) | 1);
  const int waves = hd.n <= kMaxN / 2 ? 16 : 8;
  const size_t lds = sizeof(uint32_t) * (size_t)waves * bins + 2 * sizeof(uint16_t) * (size_t)((hd.n + 1) & ~1);
  constexpr size_t kMaxLds = 158 * 1024;
  if (lds > kMaxLds) return hipErrorInvalidValue;
  static LdsLimit limit;
  const hipError_t e = limit.set(reinterpret_cast<const void *>(&forest_train_k), (int)kMaxLds);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(forest_train_k, dim3((unsigned)hd.n_trees), dim3(64 * waves), lds, s, dd, rank,
                     val, nd, y, nodes, pack, aux, n_nodes, bins);
  return hipGetLastError();
}

// Where the direct kernel is the faster one. The staged one searches every feature's distinct
// values (rank_steps loads one after the other) before its walks, which are then cheaper; a
// walk takes about log2 n steps. Times of a call (us, direct / staged, n = 512 unless said):
//   up to 8 wavefronts per compute unit, or as many as the features' values in LDS leave
//   room for, latency counts: 65,536 configurations, 20 features of 58 steps: 1 tree 13 / 18,
//   8 21 / 25, 16 32 / 33, 64 100 / 86; 24 features of 88: 16 trees 32 / 38, 32 57 / 55; 5 of
//   32: 8 18 / 18, 16 30 / 27; 40 of 400: 64 135 / 153, 112 222 / 222; 24 of 78 at n = 24, 32
//   trees 27 / 33;
//   with more of them the loads of the walks do: 1,048,576 configurations, 20 features: 2 trees
//   91 / 101, 4 108 / 110, 8 143 / 127; 262,144: 2 27 / 26, 4 33 / 29; 65,536 of 120 features of
//   480 steps: 16 trees 109 / 117, 32 171 / 139; few features leave room for more wavefronts:
//   1,048,576 of 5 features: 8 trees 59 / 85, 16 103 / 122.
// A single configuration reads one path of each tree, where staging reads the whole trees: n =
// 4096, 2,000 trees 2.5 / 4.0 ms (n = 512 1.5 / 1.35).
bool forest_direct(int64_t M, const ForestDesc &hd, int rank_steps, int cus) {
  if (M == 1 && hd.n >= 3072) return true;
  const int64_t walks = (int64_t)hd.n_trees * (32 - __builtin_clz((unsigned)hd.n));
  const int64_t lds = (int64_t)sizeof(double) * 64 * hd.F + sizeof(ForestDesc) + sizeof(CotCols);
  const int64_t waves = std::min<int64_t>(8, 160 * 1024 / lds);
  if (M <= 64 * waves * cus) return 2 * walks <= 5 * (int64_t)rank_steps;
  return 20 * walks <= 7 * (int64_t)rank_steps || hd.n_trees * hd.F <= 48;
}

hipError_t launch_forest_predict(const ForestDesc *dd, const ForestDesc &hd, const ForestNode *nodes,
                                 const ForestTrees &tr,
                                 const CotCols &cols, int64_t M, const float *ei,
                                 const uint8_t *mask, float eps_f, float *p, float *acq, int cus,
                                 hipStream_t s) {
  if (M <= 0) return hipSuccess;
  if (cus < 1) return hipErrorInvalidValue;
  if (forest_direct(M, hd, tr.rank_steps, cus)) {
    hipLaunchKernelGGL(forest_predict_direct_k, dim3((unsigned)((M + 63) / 64)), dim3(64),
                       sizeof(double) * 64 * (size_t)hd.F, s, dd, nodes, cols, M, ei, mask, eps_f,
                       p, acq);
    return hipGetLastError();
  }
  // Every workgroup loads the trees, so it takes as many configurations as the LDS beside
  // them holds the ranks of, and fewer only where that would leave compute units idle.
  int waves = forest_predict_waves(hd.F);
  while (waves > 4 && M < (int64_t)64 * waves * cus) waves >>= 1;
  const size_t lds = sizeof(uint64_t) * tr.tree_words + (size_t)waves * hd.F * 64 * sizeof(uint16_t);
  if (lds > kForestLds) return hipErrorInvalidValue;
  static LdsLimit limit;
  const hipError_t e = limit.set(reinterpret_cast<const void *>(&forest_predict_k), (int)kForestLds);
  if (e != hipSuccess) return e;
  const int64_t blocks = std::min<int64_t>((M + 64 * waves - 1) / (64 * waves), cus);
  hipLaunchKernelGGL(forest_predict_k, dim3((unsigned)blocks), dim3(64 * waves), lds, s, dd, tr.pack,
                     tr.n_nodes, tr.lofs, tr.bstart, tr.nbatch, (int)tr.tree_words, tr.val, tr.nd,
                     cols, M, ei, mask, eps_f, p, acq);
  return hipGetLastError();
}

}  // namespace bgp
