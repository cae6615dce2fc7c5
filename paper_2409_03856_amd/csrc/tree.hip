// Tree drafting step on gfx950 (Sec. 4, hardware-friendly tree building): from the sparse
// model's logits at the Wc current leaves of each tree, keep the W expansions (parent leaf,
// token) of largest cumulative log-likelihood, ties to the lower parent slot, then the lower
// token id; the new leaves come out best first.
//
// Only a leaf's W most likely tokens can be among the W best expansions (the parent's
// cumulative value is common to its tokens), and within a leaf the order of log-likelihoods is
// the order of the raw logits. A candidate is a 64-bit key that orders (logit descending, token
// ascending): the logit's bits mapped to an order-preserving unsigned value above the
// complemented token id. Keys of one row are distinct; 0 marks an empty entry.
//
//  tree_topw_kernel    grid (segments, B * Wc): each workgroup reads one segment of 2048 or 4096
//                      logits of one leaf's row, every thread a contiguous run of 8 or 16 (all
//                      loads in flight). Lists of 4 and 8: W rounds of a DPP wave maximum over the
//                      lanes' largest remaining values give each wave's W best (the lowest lane
//                      wins a tie, so the lowest token does); one wave ranks the four lists by
//                      counting. Lists of 16: the keys above a bound from group maxima, ranked by
//                      counting. The softmax statistics (max, sum of exp((v - max) / T) in fp64)
//                      merge on the common maximum.
//  tree_select_kernel  one workgroup per tree, one wave per leaf: the segment statistics merge on
//                      the common maximum into log-likelihood (v - max) / T - log(sum), W rounds of
//                      a DPP wave maximum over the segment lists' heads give the leaf's W best
//                      tokens, and the Wc x W scored candidates are ranked by counting.
//
// Bound: two launches of short dependent chains (a 4 x 128256 step reads 2 MB). Lists are as long
// as the class of W (4, 8 or 16), so that a narrow tree pays for its own width only: W = 4 takes 5.2
// and 4.8 us there (8.9 and 8.9 with lists of 16, per-pass group bounds and a merge of the statistics
// per butterfly step). Eight trees of 16 leaves with W = 16 take 68 us (88 with passes of a running
// list, 128 with wave rounds).
#include <math.h>

#include "common.h"
#include "kernels.h"
#include "profile.h"
#include "softmax.h"

namespace sirius {
namespace {

constexpr int kTopThreads = 256;
constexpr int kTopWaves = kTopThreads / kWave;
constexpr int kKW = 16;          // tree width and current-leaf limit
constexpr int kShortRow = 64 * kTopThreads * 8;  // rows of at most 64 segments of 8 logits per thread

__device__ __forceinline__ uint32_t ordered_bits(float v) {
  const uint32_t u = __float_as_uint(v);
  return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}
__device__ __forceinline__ float from_ordered(uint32_t o) {
  return __uint_as_float((o & 0x80000000u) ? (o & 0x7fffffffu) : ~o);
}
// larger key = larger logit, then lower token
__device__ __forceinline__ uint64_t ordered_key(uint32_t o, int i) {
  return ((uint64_t)o << 32) | (uint64_t)(~(uint32_t)i);
}
__device__ __forceinline__ int key_token(uint64_t k) { return (int)(~(uint32_t)k); }
__device__ __forceinline__ float key_value(uint64_t k) { return from_ordered((uint32_t)(k >> 32)); }

// v = max(v, v moved by one DPP step); rows outside ROWS keep v
template <int CTRL, int ROWS>
__device__ __forceinline__ uint64_t max_dpp(uint64_t v) {
  const int lo = (int)(uint32_t)v, hi = (int)(uint32_t)(v >> 32);
  const uint32_t olo = (uint32_t)__builtin_amdgcn_update_dpp(lo, lo, CTRL, ROWS, 0xf, false);
  const uint32_t ohi = (uint32_t)__builtin_amdgcn_update_dpp(hi, hi, CTRL, ROWS, 0xf, false);
  const uint64_t o = ((uint64_t)ohi << 32) | olo;
  return o > v ? o : v;
}

// Maximum over the 64 lanes, returned to every lane; all lanes must be active. Swaps within
// quads, rotations by 4 and 8 within rows of 16, then row 0's and row 1's results broadcast
// into the rows above: lane 63 ends with the maximum.
__device__ __forceinline__ uint64_t wave_max_u64(uint64_t v) {
  v = max_dpp<0xB1, 0xF>(v);   // quad_perm [1, 0, 3, 2]
  v = max_dpp<0x4E, 0xF>(v);   // quad_perm [2, 3, 0, 1]
  v = max_dpp<0x124, 0xF>(v);  // row_ror:4
  v = max_dpp<0x128, 0xF>(v);  // row_ror:8
  v = max_dpp<0x142, 0xA>(v);  // row_bcast:15 into rows 1 and 3
  v = max_dpp<0x143, 0xC>(v);  // row_bcast:31 into rows 2 and 3
  const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)v, 63);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(v >> 32), 63);
  return ((uint64_t)hi << 32) | lo;
}

template <int CTRL, int ROWS>
__device__ __forceinline__ uint32_t max_dpp32(uint32_t v) {
  const uint32_t o = (uint32_t)__builtin_amdgcn_update_dpp((int)v, (int)v, CTRL, ROWS, 0xf, false);
  return o > v ? o : v;
}

// The same for 32-bit values.
__device__ __forceinline__ uint32_t wave_max_u32(uint32_t v) {
  v = max_dpp32<0xB1, 0xF>(v);
  v = max_dpp32<0x4E, 0xF>(v);
  v = max_dpp32<0x124, 0xF>(v);
  v = max_dpp32<0x128, 0xF>(v);
  v = max_dpp32<0x142, 0xA>(v);
  v = max_dpp32<0x143, 0xC>(v);
  return (uint32_t)__builtin_amdgcn_readlane((int)v, 63);
}

// Softmax statistics of 64 lanes: the common maximum, and the sums brought to it and added in a
// fixed butterfly order. A sum of 0 is an empty part (its maximum is -infinity or irrelevant).
__device__ __forceinline__ void wave_stats(float& m, double& s, float c) {
  float mm = m;
#pragma unroll
  for (int k = 1; k < kWave; k <<= 1) mm = fmaxf(mm, __shfl_xor(mm, k, kWave));
  double t = s > 0.0 ? s * (double)exp2f((m - mm) * c) : 0.0;
#pragma unroll
  for (int k = 1; k < kWave; k <<= 1) t += __shfl_xor(t, k, kWave);
  m = mm;
  s = t;
}

typedef float f32x4_unaligned_t __attribute__((ext_vector_type(4), aligned(4)));

__device__ __forceinline__ uint64_t shfl_xor_u64(uint64_t v, int m) {
  const uint32_t lo = __shfl_xor((uint32_t)v, m, kWave);
  const uint32_t hi = __shfl_xor((uint32_t)(v >> 32), m, kWave);
  return ((uint64_t)hi << 32) | lo;
}

// The workgroup's W best of E keys per thread (0 = none), best first, into s_best[0 .. kKW) with 0 past
// the last. The threads form G interleaved groups (G the power of two at or above W): the W best are at
// least the W-th largest group maximum, so only the keys at or above that bound (usually a handful)
// are gathered and ranked by counting.
constexpr int kRankBatch = 16;  // LDS reads in flight per step of a rank-by-counting loop
template <int E>
__device__ void bound_best(const uint64_t (&key)[E], int W, uint64_t* __restrict__ s_best) {
  __shared__ uint64_t s_cand[kTopThreads * E + kRankBatch];
  __shared__ uint64_t s_g[kTopWaves * kKW];  // group maxima per wave
  __shared__ uint64_t s_bound;
  __shared__ int s_scan[kTopWaves];
  const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid >> 6;
  int G = 1;
  while (G < W) G <<= 1;
  uint64_t gk = 0;
#pragma unroll
  for (int j = 0; j < E; ++j) gk = key[j] > gk ? key[j] : gk;
  for (int k = G; k < kWave; k <<= 1) {
    const uint64_t o = shfl_xor_u64(gk, k);
    gk = o > gk ? o : gk;
  }
  if (lane < G) s_g[wave * kKW + lane] = gk;
  if (tid == 0) s_bound = 0;
  if (tid < kKW) s_best[tid] = 0;
  __syncthreads();
  if (tid < G) {
    uint64_t gm[kKW];
#pragma unroll
    for (int g = 0; g < kKW; ++g) {
      uint64_t x = 0;
#pragma unroll
      for (int w = 0; w < kTopWaves; ++w) {
        const uint64_t y = s_g[w * kKW + g];
        x = y > x ? y : x;
      }
      gm[g] = g < G ? x : 0;
    }
    uint64_t mine = 0;
#pragma unroll
    for (int g = 0; g < kKW; ++g) mine = g == tid ? gm[g] : mine;
    int r = 0;
#pragma unroll
    for (int g = 0; g < kKW; ++g) r += gm[g] > mine;
    if (mine != 0 && r == W - 1) s_bound = mine;
  }
  __syncthreads();
  const uint64_t bound = s_bound;
  int n = 0, ncand = 0;
#pragma unroll
  for (int j = 0; j < E; ++j) n += (key[j] != 0 && key[j] >= bound);
  int pos = block_exclusive_scan_256(n, s_scan, &ncand);
#pragma unroll
  for (int j = 0; j < E; ++j)
    if (key[j] != 0 && key[j] >= bound) s_cand[pos++] = key[j];
  const int npad = (ncand + kRankBatch - 1) / kRankBatch * kRankBatch;
  if (tid < npad - ncand) s_cand[ncand + tid] = 0;  // empty: never counted as larger
  __syncthreads();
  for (int i = tid; i < ncand; i += kTopThreads) {
    const uint64_t k0 = s_cand[i];
    int r = 0;
    for (int j = 0; j < npad; j += kRankBatch) {
      uint64_t buf[kRankBatch];
#pragma unroll
      for (int q = 0; q < kRankBatch; ++q) buf[q] = s_cand[j + q];
#pragma unroll
      for (int q = 0; q < kRankBatch; ++q) r += (int)(buf[q] > k0);
    }
    if (r < W) s_best[r] = k0;
  }
  __syncthreads();
}

// E logits per thread; lists of KW entries (W <= KW).
template <int E, int KW>
__global__ __launch_bounds__(kTopThreads) void tree_topw_kernel(
    const float* __restrict__ logits, int V, int W, float c, float* __restrict__ rm,
    double* __restrict__ rs, uint64_t* __restrict__ rk) {
  // one list per wave, ranked into one at the end; the longest lists are formed by the workgroup at once
  constexpr bool kBound = KW == kKW;
  __shared__ uint64_t s_c[kBound ? KW : kTopWaves * KW];
  __shared__ float s_m[kTopWaves];
  __shared__ double s_s[kTopWaves];
  const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid >> 6;
  const int split = blockIdx.x, row = blockIdx.y, splits = gridDim.x;
  const int e0 = split * kTopThreads * E + tid * E;
  const float* L = logits + (size_t)row * V;
  float v[E];
  if (e0 + E <= V) {
    // the row starts on a 16-byte boundary only when V % 4 == 0: loads of four with 4-byte alignment
#pragma unroll
    for (int g = 0; g < E / 4; ++g) {
      const f32x4_unaligned_t x = *reinterpret_cast<const f32x4_unaligned_t*>(L + e0 + 4 * g);
#pragma unroll
      for (int j = 0; j < 4; ++j) v[4 * g + j] = x[j];
    }
  } else {
#pragma unroll
    for (int j = 0; j < E; ++j) v[j] = (e0 + j < V) ? L[e0 + j] : -INFINITY;
  }
  if (!kBound && tid < kTopWaves * KW) s_c[tid] = 0;
  // softmax statistics of the thread: exps summed pairwise in fp32 (at most 16 terms, each <= 1)
  float m = -INFINITY;
#pragma unroll
  for (int j = 0; j < E; ++j) m = fmaxf(m, v[j]);
  float t[E / 4];
#pragma unroll
  for (int g = 0; g < E / 4; ++g)
    t[g] = (exp2_nonpos((v[4 * g] - m) * c) + exp2_nonpos((v[4 * g + 1] - m) * c)) +
           (exp2_nonpos((v[4 * g + 2] - m) * c) + exp2_nonpos((v[4 * g + 3] - m) * c));
#pragma unroll
  for (int k = 1; k < E / 4; k <<= 1)
#pragma unroll
    for (int g = 0; g < E / 4; g += 2 * k) t[g] += t[g + k];
  double s = m > -INFINITY ? (double)t[0] : 0.0;  // -inf logits add nothing
  const size_t at = (size_t)row * splits + split;
  if constexpr (kBound) {
    uint64_t key[E];
#pragma unroll
    for (int j = 0; j < E; ++j) key[j] = e0 + j < V ? ordered_key(ordered_bits(v[j]), e0 + j) : 0;
    bound_best<E>(key, W, s_c);
    if (tid < KW) rk[at * KW + tid] = s_c[tid];
  } else {
    uint32_t o[E], lm = 0;
#pragma unroll
    for (int j = 0; j < E; ++j) {
      o[j] = (e0 + j < V) ? ordered_bits(v[j]) : 0u;
      lm = o[j] > lm ? o[j] : lm;
    }
    __syncthreads();
    // the wave's W best, best first
    for (int r = 0; r < W; ++r) {
      const uint32_t best = wave_max_u32(lm);
      if (best == 0u) break;  // uniform: nothing left
      const bool win = lane == __builtin_ctzll(__ballot(lm == best));
      int jj = 0;
#pragma unroll
      for (int j = E - 1; j >= 0; --j) jj = o[j] == best ? j : jj;
      if (win) s_c[wave * KW + r] = ordered_key(best, e0 + jj);
      uint32_t next = 0;
#pragma unroll
      for (int j = 0; j < E; ++j) {
        o[j] = (win && j == jj) ? 0u : o[j];
        next = o[j] > next ? o[j] : next;
      }
      lm = next;
    }
  }
  wave_stats(m, s, c);
  if (lane == 0) {
    s_m[wave] = m;
    s_s[wave] = s;
  }
  __syncthreads();
  if (wave != 0) return;
  if constexpr (!kBound) {
    // rank the four lists by counting (non-empty keys are distinct)
    constexpr int kN = kTopWaves * KW;
    const uint64_t key = lane < kN ? s_c[lane] : 0;
    int rank = 0, n = 0;
#pragma unroll
    for (int i = 0; i < kN; ++i) {
      const uint64_t k = s_c[i];
      rank += (int)(k > key);
      n += (int)(k != 0);
    }
    if (key != 0 && rank < W) rk[at * KW + rank] = key;
    if (lane >= n && lane < KW) rk[at * KW + lane] = 0;
    if (lane < KW && lane >= W) rk[at * KW + lane] = 0;
  }
  if (lane == 0) {
    float am = s_m[0];
#pragma unroll
    for (int w = 1; w < kTopWaves; ++w) am = fmaxf(am, s_m[w]);
    double as = 0.0;
#pragma unroll
    for (int w = 0; w < kTopWaves; ++w)
      if (s_s[w] > 0.0) as += s_s[w] * (double)exp2f((s_m[w] - am) * c);
    rm[at] = am;
    rs[at] = as;
  }
}

template <int KW>
__global__ __launch_bounds__(kKW * kWave) void tree_select_kernel(
    int Wc, int W, int splits, float c, float inv_t, const float* __restrict__ rm,
    const double* __restrict__ rs, const uint64_t* __restrict__ rk,
    const float* __restrict__ cum_in, int32_t* __restrict__ tokens, int32_t* __restrict__ parents,
    float* __restrict__ cum_out) {
  __shared__ double s_sc[kKW * KW];  // each leaf's W best, scored: [leaf][rank]
  __shared__ int s_tk[kKW * KW];
  const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid >> 6;
  const int b = blockIdx.x;
  {  // one wave per leaf, one lane per segment (segments lane, lane + 64, ..)
    const size_t row = (size_t)b * Wc + wave;
    const uint64_t* lists = rk + row * splits * KW;
    uint64_t lst[KW];  // the lane's best, best first (0 = empty)
#pragma unroll
    for (int p = 0; p < KW; ++p) lst[p] = lane < splits ? lists[(size_t)lane * KW + p] : 0;
    float m = lane < splits ? rm[row * splits + lane] : -INFINITY;
    double s = lane < splits ? rs[row * splits + lane] : 0.0;
    const float base = cum_in != nullptr ? cum_in[row] : 0.f;
    for (int sp = lane + kWave; sp < splits; sp += kWave) {  // rows of more than 64 segments
      const float om = rm[row * splits + sp];
      const double os = rs[row * splits + sp];
      const float mm = fmaxf(m, om);
      double ns = s > 0.0 ? s * (double)exp2f((m - mm) * c) : 0.0;
      if (os > 0.0) ns += os * (double)exp2f((om - mm) * c);
      m = mm;
      s = ns;
      for (int q = 0; q < KW; ++q) {
        uint64_t x = lists[(size_t)sp * KW + q];
#pragma unroll
        for (int p = 0; p < KW; ++p) {  // insert: the rest moves down
          const uint64_t y = lst[p];
          lst[p] = x > y ? x : y;
          x = x > y ? y : x;
        }
      }
    }
    wave_stats(m, s, c);
    const double lse = log(s);  // log of sum exp((v - m) / T)
    // the leaf's W best: W rounds of a wave maximum over the list heads
    uint64_t mine = 0;
    for (int r = 0; r < W; ++r) {
      const uint64_t best = wave_max_u64(lst[0]);
      const bool win = best != 0 && lst[0] == best;  // non-empty keys are distinct
#pragma unroll
      for (int p = 0; p < KW - 1; ++p) lst[p] = win ? lst[p + 1] : lst[p];
      lst[KW - 1] = win ? 0 : lst[KW - 1];
      mine = lane == r ? best : mine;
    }
    if (lane < W) {
      const double lp = ((double)key_value(mine) - (double)m) * (double)inv_t - lse;
      s_sc[wave * KW + lane] = mine != 0 ? (double)base + lp : -INFINITY;
      s_tk[wave * KW + lane] = mine != 0 ? key_token(mine) : -1;
    }
  }
  __syncthreads();
  // the W best of the Wc x W: valid first, larger score, lower parent, lower token
  const int m2 = Wc * W;
  for (int i = tid; i < m2; i += blockDim.x) {
    const int leaf = i / W, r0 = i - leaf * W;
    const double sc = s_sc[leaf * KW + r0];
    const int tk = s_tk[leaf * KW + r0];
    const bool ok = tk >= 0;
    int r = 0;
    for (int lj = 0; lj < Wc; ++lj) {
      double so[KW];
      int to[KW];
#pragma unroll
      for (int rj = 0; rj < KW; ++rj) {
        so[rj] = s_sc[lj * KW + rj];
        to[rj] = s_tk[lj * KW + rj];
      }
#pragma unroll
      for (int rj = 0; rj < KW; ++rj) {
        const bool okj = to[rj] >= 0;
        const bool tie_lower = (lj < leaf) | ((lj == leaf) & ((to[rj] < tk) | ((to[rj] == tk) & (rj < r0))));
        const bool better = (okj & !ok) | ((okj == ok) & ((so[rj] > sc) | ((so[rj] == sc) & tie_lower)));
        r += (int)((rj < W) & better);
      }
    }
    if (r < W) {
      tokens[(size_t)b * W + r] = ok ? tk : -1;
      parents[(size_t)b * W + r] = ok ? leaf : -1;
      cum_out[(size_t)b * W + r] = (float)sc;
    }
  }
}

int list_len(int W) { return W <= 4 ? 4 : (W <= 8 ? 8 : kKW); }

}  // namespace

TreeBuildLayout tree_build_layout(int B, int Wc, int W, int V) {
  TreeBuildLayout L{};
  const int rows = std::max(1, B * Wc);
  // eight logits per thread (twice the workgroups) while a leaf's segments fit the select's lanes; the
  // longest lists cost a workgroup the same whatever it reads
  L.splits = ceil_div(V, kTopThreads * (V <= kShortRow && list_len(W) < kKW ? 8 : 16));
  const size_t n = (size_t)rows * L.splits;
  Carve c;
  L.rm = c.take(n * sizeof(float));
  L.rs = c.take(n * sizeof(double));
  L.rk = c.take(n * list_len(W) * sizeof(uint64_t));
  L.total = c.off;
  return L;
}

hipError_t launch_tree_build(const float* logits, int B, int Wc, int V, const float* cum_ll, int W,
                             float temperature, int32_t* tokens, int32_t* parents,
                             float* cum_out, char* ws, const TreeBuildLayout& L,
                             hipStream_t stream) {
  if (W < 1 || W > kKW || Wc < 1 || Wc > kKW) return hipErrorInvalidValue;
  float* rm = reinterpret_cast<float*>(ws + L.rm);
  double* rs = reinterpret_cast<double*>(ws + L.rs);
  uint64_t* rk = reinterpret_cast<uint64_t*>(ws + L.rk);
  const float c = (float)(1.4426950408889634 / (double)temperature);
  const dim3 grid(L.splits, B * Wc);
  {
    ProfScope prof("tree_topw", stream);
#define SIRIUS_TOPW(E, KW) \
  klaunch((tree_topw_kernel<E, KW>), grid, kTopThreads, 0, stream, logits, V, W, c, rm, rs, rk)
    // Wave rounds up to lists of 8, group bounds for lists of 16: at 8 x 16 leaves of 128256 tokens the
    // rounds take 95 us for W = 16 and the bounds 51.
    if (W > 8) {
      SIRIUS_TOPW(16, 16);
    } else if (W > 4) {
      if (V <= kShortRow) SIRIUS_TOPW(8, 8);
      else SIRIUS_TOPW(16, 8);
    } else {
      if (V <= kShortRow) SIRIUS_TOPW(8, 4);
      else SIRIUS_TOPW(16, 4);
    }
#undef SIRIUS_TOPW
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  ProfScope prof("tree_select", stream);
  const float inv_t = (float)(1.0 / temperature);
  if (W <= 4)
    klaunch(tree_select_kernel<4>, B, Wc * kWave, 0, stream, Wc, W, L.splits, c, inv_t, rm, rs, rk, cum_ll,
            tokens, parents, cum_out);
  else if (W <= 8)
    klaunch(tree_select_kernel<8>, B, Wc * kWave, 0, stream, Wc, W, L.splits, c, inv_t, rm, rs, rk, cum_ll,
            tokens, parents, cum_out);
  else
    klaunch(tree_select_kernel<16>, B, Wc * kWave, 0, stream, Wc, W, L.splits, c, inv_t, rm, rs, rk, cum_ll,
            tokens, parents, cum_out);
  return hipGetLastError();
}

}  // namespace sirius
