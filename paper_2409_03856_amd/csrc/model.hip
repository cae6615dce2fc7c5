// A small Llama-style decoder built from the library's kernels, and the Sirius generation
// loop (Algorithm 1) over it with every decision kept on the device.
//
//  embed_kernel        h[i] = E[token_i] (bf16 rows widened; an id outside [0, V) gives 0)
//  linear_kernel       one token: y[j] = x . W[j] (+ resid[j]), x staged in LDS, one wave per
//                      output row (W row-major [N][K] bf16)
//  norm_qkv_kernel     one token: RMSNorm of the row as it is staged (the same sums, in the same
//                      order, as rmsnorm_vec_kernel, so bit for bit its result), then the
//                      products of up to three matrices in one launch: q = xn Wq^T (fp32),
//                      k = xn Wk^T and v = xn Wv^T (bf16) -- a layer's attention inputs, or the
//                      final norm and the LM head (q only)
//  linear_pair_kernel  both for two tokens at small layers. Other chunks run in linear.hip
//  draft_tail_kernel   the sparse model's greedy draft: argmax of one logit row (lowest index
//                      on ties) into the chunk buffer, and the cache position advanced by one
//                      (wound back by n - 1 after the last draft, so the full model's pass
//                      starts at the period's first position)
//  period_tail_kernel  after the check: the rollback to P + min(j + 1, n), the accepted
//                      drafts and the corrected token appended to the output, and the next
//                      period's first input (the corrected token, or the last draft)
//
// One period is a fixed sequence of launches on one stream -- n sparse passes, one full pass
// over the n-token chunk, the check, the tail -- with the positions, drafts, acceptance and
// output count living in device memory, so periods run back to back without a host round
// trip.
#include "common.h"
#include "kernels.h"
#include "profile.h"

namespace sirius {
namespace {

constexpr int kLinThreads = 256;
constexpr int kLinWaves = kLinThreads / kWave;
constexpr int kLinMaxK = 8192;  // floats of x staged per launch
constexpr int kLinMaxPartK = 512;  // widest row summed from FFN partials on the way in
constexpr int kPartBlocks = 128;   // workgroups that read the FFN's partials at most
constexpr int kTailThreads = 1024;
static_assert(kLinMaxPartK <= 4 * kLinThreads && kLinMaxPartK / 4 * 16 <= kLinMaxK / 4, "one column per thread; LDS");

// Where the row of a one-token projection comes from (norm_qkv_kernel).
struct StepRow {
  const float* x;        // kSrcRow: the row; kSrcPartials: the residual
  const int32_t* token;  // kSrcToken
  const uint2* embed;
  int V;
  const float* logits;   // kSrcToken after a draft: the previous step's logits, else null
  int32_t* seq;
  int slot;
  int32_t* cache_pos;
  int32_t* trace_drafted;
  const float* part;     // kSrcPartials: [nseg][K]
  int nseg;
  float* h_out;          // kSrcToken, kSrcPartials: the row, for the residuals that follow
};
constexpr int kSrcRow = 0, kSrcToken = 1, kSrcPartials = 2;

__global__ __launch_bounds__(256) void embed_kernel(const int32_t* __restrict__ tokens, int n,
                                                    const uint4* __restrict__ E, int d8, int V,
                                                    float* __restrict__ out) {
  const int i = blockIdx.x;
  if (i >= n) return;
  const int tok = tokens[i];
  const bool ok = tok >= 0 && tok < V;
  float4* o = reinterpret_cast<float4*>(out + (size_t)i * d8 * 8);
  for (int c = threadIdx.x; c < d8; c += blockDim.x) {
    const uint4 w = ok ? E[(size_t)tok * d8 + c] : make_uint4(0u, 0u, 0u, 0u);
    o[2 * c] = make_float4(bf16_lo(w.x), bf16_hi(w.x), bf16_lo(w.y), bf16_hi(w.y));
    o[2 * c + 1] = make_float4(bf16_lo(w.z), bf16_hi(w.z), bf16_lo(w.w), bf16_hi(w.w));
  }
}

// Rows j = blockIdx.x * 4 + wave, + gridDim.x * 4, ...; x in LDS.
__global__ __launch_bounds__(kLinThreads) void linear_kernel(const float* __restrict__ x,
                                                             const uint4* __restrict__ W, int K,
                                                             int N, const float* resid, float* y) {
  __shared__ float4 s_x4[kLinMaxK / 4];
  const float* xs = reinterpret_cast<const float*>(s_x4);
  const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid >> 6;
  const int k4 = K >> 2, k8 = K >> 3;
  const float4* x4 = reinterpret_cast<const float4*>(x);
  for (int e = tid; e < k4; e += kLinThreads) s_x4[e] = x4[e];
  __syncthreads();
  for (int j = blockIdx.x * kLinWaves + wave; j < N; j += gridDim.x * kLinWaves) {
    const uint4* wr = W + (size_t)j * k8;
    float acc = 0.f;
    for (int c = lane; c < k8; c += kWave) acc = dot8(wr[c], xs + 8 * c, acc);
    const float s = wave_sum(acc);
    if (lane == 0) y[j] = (resid != nullptr) ? resid[j] + s : s;
  }
}

// Argmax over one row of V logits, lowest index on ties: (value, index) pairs reduced so
// that the larger value wins and, on equal values, the smaller index.
__device__ __forceinline__ void better(float& v, int& i, float ov, int oi) {
  if (ov > v || (ov == v && oi < i)) {
    v = ov;
    i = oi;
  }
}

template <int THREADS>
__device__ int block_argmax(const float* __restrict__ row, int V) {
  constexpr int kAhead = 4;  // loads in flight per thread
  __shared__ float s_v[THREADS / kWave];
  __shared__ int s_i[THREADS / kWave];
  const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid >> 6;
  float bv = -INFINITY;
  int bi = INT32_MAX;
  for (int v0 = tid; v0 < V; v0 += THREADS * kAhead) {
    float x[kAhead];
#pragma unroll
    for (int u = 0; u < kAhead; ++u) x[u] = v0 + u * THREADS < V ? row[v0 + u * THREADS] : -INFINITY;
#pragma unroll
    for (int u = 0; u < kAhead; ++u)
      if (v0 + u * THREADS < V) better(bv, bi, x[u], v0 + u * THREADS);
  }
#pragma unroll
  for (int m = 32; m >= 1; m >>= 1) {
    const float ov = __shfl_xor(bv, m, kWave);
    const int oi = __shfl_xor(bi, m, kWave);
    better(bv, bi, ov, oi);
  }
  if (lane == 0) {
    s_v[wave] = bv;
    s_i[wave] = bi;
  }
  __syncthreads();
  bv = s_v[0];
  bi = s_i[0];
  for (int w = 1; w < THREADS / kWave; ++w) better(bv, bi, s_v[w], s_i[w]);
  return bi == INT32_MAX ? 0 : bi;  // a row of NaNs only
}

// Output rows j of the three products in one range: [0, Nq) of Wq into yq (fp32), then
// [Nq, Nq + Nkv) of Wk and [Nq + Nkv, Nq + 2 Nkv) of Wv into yk, yv (bf16). The row x is formed
// in every workgroup (SRC, see StepRow; workgroup 0 writes it to h_out), then normalised: each
// thread sums the squares of its float4s tid + 256 u as rmsnorm_vec_kernel does, the wave sums go
// through LDS, and each thread scales its float4s into LDS.
//   kSrcRow       x is the row given.
//   kSrcToken     x is a token's embedding. The token is given, or (logits != nullptr) it is the
//                 argmax of the previous step's logits, which every workgroup finds for itself;
//                 workgroup 0 then does what draft_tail_kernel does.
//   kSrcPartials  x = resid + the batch-1 FFN's segment partials, added in reduce_kernel's order
//                 (16 groups of every 16th row, then the groups), so the same bits.
// The last two save a dependent launch of 2-4 us each at the loop's small decoder, where they add
// 1-2 us to this one: two periods of 16 drafts on the 2-layer, 256-wide decoder 1827 -> 1607 us.
constexpr int kPartGroups = 16;  // reduce_kernel's groups of partial rows

template <int SRC>
__global__ __launch_bounds__(kLinThreads) void norm_qkv_kernel(
    StepRow in, int K, float eps, const uint4* __restrict__ Wq, int Nq,
    const uint4* __restrict__ Wk, const uint4* __restrict__ Wv, int Nkv, float* __restrict__ yq,
    uint16_t* __restrict__ yk, uint16_t* __restrict__ yv) {
  static_assert(kLinThreads == 256, "the norm's sums follow rmsnorm_vec_kernel's 256-thread layout");
  constexpr int kPer = kLinMaxK / 4 / kLinThreads;
  __shared__ float4 s_x4[kLinMaxK / 4];
  __shared__ float s_w[kLinWaves];
  const float* xs = reinterpret_cast<const float*>(s_x4);
  const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid >> 6;
  const int k4 = K >> 2, k8 = K >> 3;
  float4 v[kPer];
  if (SRC == kSrcRow) {
    const float4* x4 = reinterpret_cast<const float4*>(in.x);
#pragma unroll
    for (int u = 0; u < kPer; ++u) {
      const int e = tid + kLinThreads * u;
      v[u] = (e < k4) ? x4[e] : make_float4(0.f, 0.f, 0.f, 0.f);
    }
  } else if (SRC == kSrcToken) {
    int tok;
    if (in.logits != nullptr) {  // uniform
      tok = block_argmax<kLinThreads>(in.logits, in.V);
      if (blockIdx.x == 0 && tid == 0) {
        in.seq[in.slot] = tok;
        in.cache_pos[0] += 1;
        if (in.trace_drafted != nullptr) in.trace_drafted[in.slot - 1] = tok;
      }
    } else {
      tok = in.token[0];
    }
    const bool ok = tok >= 0 && tok < in.V;
    const uint2* row = in.embed + (size_t)(ok ? tok : 0) * k4;
#pragma unroll
    for (int u = 0; u < kPer; ++u) {
      const int e = tid + kLinThreads * u;
      const uint2 w = (ok && e < k4) ? row[e] : make_uint2(0u, 0u);
      v[u] = make_float4(bf16_lo(w.x), bf16_hi(w.x), bf16_lo(w.y), bf16_hi(w.y));
    }
  } else {
    // (group, column) pairs of kPartGroups x k4 (k4 <= 128): at most eight per thread, the loads of
    // four partial rows of every pair in flight
    constexpr int kPairs = kLinMaxPartK / 4 * kPartGroups / kLinThreads, kAhead = 4;
    const float4* p4 = reinterpret_cast<const float4*>(in.part);
    float4 s[kPairs];
#pragma unroll
    for (int k = 0; k < kPairs; ++k) s[k] = make_float4(0.f, 0.f, 0.f, 0.f);
    for (int r0 = 0; r0 < in.nseg; r0 += kPartGroups * kAhead) {
      float4 w[kAhead][kPairs];
#pragma unroll
      for (int a = 0; a < kAhead; ++a)
#pragma unroll
        for (int k = 0; k < kPairs; ++k) {
          const int pair = tid + kLinThreads * k, g = pair / k4, c = pair - g * k4;
          const int r = r0 + kPartGroups * a + g;
          w[a][k] = (g < kPartGroups && r < in.nseg) ? p4[(size_t)r * k4 + c] : make_float4(0.f, 0.f, 0.f, 0.f);
        }
#pragma unroll
      for (int a = 0; a < kAhead; ++a)
#pragma unroll
        for (int k = 0; k < kPairs; ++k) {
          s[k].x += w[a][k].x;
          s[k].y += w[a][k].y;
          s[k].z += w[a][k].z;
          s[k].w += w[a][k].w;
        }
    }
#pragma unroll
    for (int k = 0; k < kPairs; ++k) {
      const int pair = tid + kLinThreads * k;
      if (pair < kPartGroups * k4) s_x4[pair] = s[k];  // [group][column]
    }
    __syncthreads();
    v[0] = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
    for (int u = 1; u < kPer; ++u) v[u] = v[0];
    if (tid < k4) {
      float4 t = s_x4[tid];
      for (int g = 1; g < kPartGroups; ++g) {
        const float4 a = s_x4[g * k4 + tid];
        t.x += a.x;
        t.y += a.y;
        t.z += a.z;
        t.w += a.w;
      }
      const float4 r = reinterpret_cast<const float4*>(in.x)[tid];
      v[0] = make_float4(r.x + t.x, r.y + t.y, r.z + t.z, r.w + t.w);
    }
    __syncthreads();  // the partials are read: the normalised row takes their place
  }
  if (SRC != kSrcRow && blockIdx.x == 0) {
#pragma unroll
    for (int u = 0; u < kPer; ++u) {
      const int e = tid + kLinThreads * u;
      if (e < k4) reinterpret_cast<float4*>(in.h_out)[e] = v[u];
    }
  }
  float ss = 0.f;
#pragma unroll
  for (int u = 0; u < kPer; ++u) {
    ss = fmaf(v[u].x, v[u].x, ss);
    ss = fmaf(v[u].y, v[u].y, ss);
    ss = fmaf(v[u].z, v[u].z, ss);
    ss = fmaf(v[u].w, v[u].w, ss);
  }
  ss = wave_sum(ss);
  if (lane == 0) s_w[wave] = ss;
  __syncthreads();
  const float tot = ((s_w[0] + s_w[1]) + s_w[2]) + s_w[3];
  const float inv = 1.0f / sqrtf(tot / (float)K + eps);
#pragma unroll
  for (int u = 0; u < kPer; ++u) {
    const int e = tid + kLinThreads * u;
    if (e < k4) s_x4[e] = make_float4(v[u].x * inv, v[u].y * inv, v[u].z * inv, v[u].w * inv);
  }
  __syncthreads();
  const int N = Nq + 2 * Nkv;
  for (int j = blockIdx.x * kLinWaves + wave; j < N; j += gridDim.x * kLinWaves) {
    const int part = j < Nq ? 0 : (j < Nq + Nkv ? 1 : 2);  // uniform over the wave
    const int jr = part == 0 ? j : (part == 1 ? j - Nq : j - Nq - Nkv);
    const uint4* wr = (part == 0 ? Wq : (part == 1 ? Wk : Wv)) + (size_t)jr * k8;
    float acc = 0.f;
    for (int c = lane; c < k8; c += kWave) acc = dot8(wr[c], xs + 8 * c, acc);
    const float s = wave_sum(acc);
    if (lane == 0) {
      if (part == 0) yq[jr] = s;
      else (part == 1 ? yk : yv)[jr] = (uint16_t)f32_to_bf16(s);
    }
  }
}

// Two tokens' products in one launch: norm_qkv_kernel's (eps >= 0) or linear_kernel's sums for both
// rows of x, each weight read once.
constexpr int kPairMaxK = 2048;
__global__ __launch_bounds__(kLinThreads) void linear_pair_kernel(
    const float* __restrict__ x, int K, float eps, const uint4* __restrict__ Wq, int Nq,
    const uint4* __restrict__ Wk, const uint4* __restrict__ Wv, int Nkv, const float* resid, float* yq,
    uint16_t* __restrict__ yk, uint16_t* __restrict__ yv) {
  constexpr int kPer = kPairMaxK / 4 / kLinThreads;
  __shared__ float4 s_x4[2][kPairMaxK / 4];
  __shared__ float s_w[2][kLinWaves];
  const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid >> 6;
  const int k4 = K >> 2, k8 = K >> 3;
  const float4* x4 = reinterpret_cast<const float4*>(x);
  float4 v[2][kPer];
  float ss[2] = {0.f, 0.f};
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int u = 0; u < kPer; ++u) {
      const int e = tid + kLinThreads * u;
      v[i][u] = e < k4 ? x4[i * k4 + e] : make_float4(0.f, 0.f, 0.f, 0.f);
    }
  float inv[2] = {1.f, 1.f};
  if (eps >= 0.f) {  // uniform
#pragma unroll
    for (int i = 0; i < 2; ++i) {
#pragma unroll
      for (int u = 0; u < kPer; ++u) {
        ss[i] = fmaf(v[i][u].x, v[i][u].x, ss[i]);
        ss[i] = fmaf(v[i][u].y, v[i][u].y, ss[i]);
        ss[i] = fmaf(v[i][u].z, v[i][u].z, ss[i]);
        ss[i] = fmaf(v[i][u].w, v[i][u].w, ss[i]);
      }
      ss[i] = wave_sum(ss[i]);
      if (lane == 0) s_w[i][wave] = ss[i];
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const float tot = ((s_w[i][0] + s_w[i][1]) + s_w[i][2]) + s_w[i][3];
      inv[i] = 1.0f / sqrtf(tot / (float)K + eps);
    }
  }
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int u = 0; u < kPer; ++u) {
      const int e = tid + kLinThreads * u;
      if (e < k4)
        s_x4[i][e] = make_float4(v[i][u].x * inv[i], v[i][u].y * inv[i], v[i][u].z * inv[i], v[i][u].w * inv[i]);
    }
  __syncthreads();
  const float* xs0 = reinterpret_cast<const float*>(s_x4[0]);
  const float* xs1 = reinterpret_cast<const float*>(s_x4[1]);
  const int N = Nq + 2 * Nkv;
  for (int j = blockIdx.x * kLinWaves + wave; j < N; j += gridDim.x * kLinWaves) {
    const int part = j < Nq ? 0 : (j < Nq + Nkv ? 1 : 2);  // uniform over the wave
    const int jr = part == 0 ? j : (part == 1 ? j - Nq : j - Nq - Nkv);
    const uint4* wr = (part == 0 ? Wq : (part == 1 ? Wk : Wv)) + (size_t)jr * k8;
    float a0 = 0.f, a1 = 0.f;
    for (int c = lane; c < k8; c += kWave) {
      const uint4 w = wr[c];
      a0 = dot8(w, xs0 + 8 * c, a0);
      a1 = dot8(w, xs1 + 8 * c, a1);
    }
    a0 = wave_sum(a0);
    a1 = wave_sum(a1);
    if (lane < 2) {
      const float s = lane == 0 ? a0 : a1;
      if (part == 0) {
        const size_t o = (size_t)lane * Nq + jr;
        yq[o] = resid != nullptr ? resid[o] + s : s;
      } else {
        (part == 1 ? yk : yv)[(size_t)lane * Nkv + jr] = (uint16_t)f32_to_bf16(s);
      }
    }
  }
}

__global__ __launch_bounds__(kTailThreads) void draft_tail_kernel(
    const float* __restrict__ logits, int V, int32_t* __restrict__ seq, int slot,
    int32_t* __restrict__ cache_pos, int pos_delta, int32_t* __restrict__ trace_drafted) {
  const int tok = block_argmax<kTailThreads>(logits, V);
  if (threadIdx.x == 0) {
    seq[slot] = tok;
    cache_pos[0] += pos_delta;
    if (trace_drafted != nullptr) trace_drafted[slot - 1] = tok;
  }
}

__global__ void period_tail_kernel(int32_t* __restrict__ seq, int n,
                                   const int32_t* __restrict__ accept_len,
                                   const int32_t* __restrict__ next_token,
                                   int32_t* __restrict__ cache_pos, int32_t* __restrict__ out,
                                   int32_t* __restrict__ out_count, int out_cap,
                                   int32_t* __restrict__ tr_accept, int32_t* __restrict__ tr_next) {
  if (threadIdx.x != 0) return;
  int j = accept_len[0];
  j = j < 0 ? 0 : (j > n ? n : j);
  const int nxt = next_token[0];
  cache_pos[0] += (j + 1 < n) ? j + 1 : n;
  int c = out_count[0];
  for (int i = 1; i <= j; ++i)
    if (c >= 0 && c < out_cap) out[c++] = seq[i];
  if (j < n) {
    if (c >= 0 && c < out_cap) out[c++] = nxt;
    seq[0] = nxt;
  } else {
    seq[0] = seq[n];
  }
  out_count[0] = c;
  if (tr_accept != nullptr) tr_accept[0] = j;
  if (tr_next != nullptr) tr_next[0] = (j < n) ? nxt : -1;
}

}  // namespace

hipError_t launch_embed(const int32_t* tokens, int n, const uint16_t* E, int d, int V, float* out,
                        hipStream_t s) {
  ProfScope prof("embed", s);
  klaunch(embed_kernel, n, 256, 0, s, tokens, n, reinterpret_cast<const uint4*>(E), d / 8, V, out);
  return hipGetLastError();
}

hipError_t launch_norm_qkv(const StepSource& src, int K, float eps, const uint16_t* Wq, int Nq,
                           const uint16_t* Wk, const uint16_t* Wv, int Nkv, float* yq, uint16_t* yk,
                           uint16_t* yv, hipStream_t s) {
  if ((K & 7) != 0 || K > kLinMaxK || Nq < 1 || Nkv < 0 ||
      (Nkv > 0 && (Wk == nullptr || Wv == nullptr || yk == nullptr || yv == nullptr)) ||
      (src.part != nullptr && K > kLinMaxPartK))
    return hipErrorInvalidValue;
  ProfScope prof("norm_qkv", s);
  const StepRow in{src.x, src.token, reinterpret_cast<const uint2*>(src.embed), src.V, src.logits, src.seq,
                   src.slot, src.cache_pos, src.trace_drafted, src.part, src.nseg, src.h_out};
  const int grid = std::min(ceil_div(Nq + 2 * Nkv, kLinWaves), src.part != nullptr ? kPartBlocks : 2048);
  const uint4* q4 = reinterpret_cast<const uint4*>(Wq);
  const uint4* k4 = reinterpret_cast<const uint4*>(Wk);
  const uint4* v4 = reinterpret_cast<const uint4*>(Wv);
  if (src.part != nullptr)
    klaunch(norm_qkv_kernel<kSrcPartials>, grid, kLinThreads, 0, s, in, K, eps, q4, Nq, k4, v4, Nkv, yq, yk, yv);
  else if (src.embed != nullptr)
    klaunch(norm_qkv_kernel<kSrcToken>, grid, kLinThreads, 0, s, in, K, eps, q4, Nq, k4, v4, Nkv, yq, yk, yv);
  else
    klaunch(norm_qkv_kernel<kSrcRow>, grid, kLinThreads, 0, s, in, K, eps, q4, Nq, k4, v4, Nkv, yq, yk, yv);
  return hipGetLastError();
}

// What every workgroup of the launch reads for itself comes from L2 at about 8 TB/s over the chip:
// at most 1.5 us of partials and 1 us of logits. The kPartBlocks workgroups that take partials also
// take all N rows, where the separate sum (3-4 us) leaves up to 2048 workgroups to them: at most three
// rows per wave. At 256 x 688 the fold saves 1.5 us per projection of 300-1000 rows, 0 at 2000 and
// costs 3 at 8000 and 10 at 16000; at 512 x 1024 (2 us of partials) it saves nothing at 300.
bool step_takes_partials(int K, int nseg, int N) {
  return K <= kLinMaxPartK && N <= 3 * kPartBlocks * kLinWaves &&
         (size_t)kPartBlocks * nseg * K * sizeof(float) <= (size_t)12 << 20;
}
bool step_takes_logits(int V, int N) {
  return (size_t)std::min(ceil_div(N, kLinWaves), 2048) * V * sizeof(float) <= (size_t)8 << 20;
}

hipError_t launch_linear(const float* x, const uint16_t* W, int K, int N, const float* resid, float* y,
                         hipStream_t s) {
  if ((K & 7) != 0 || K > kLinMaxK) return hipErrorInvalidValue;
  ProfScope prof("linear", s);
  klaunch(linear_kernel, std::min(ceil_div(N, kLinWaves), 2048), kLinThreads, 0, s, x,
          reinterpret_cast<const uint4*>(W), K, N, resid, y);
  return hipGetLastError();
}

// Up to two million weights the launch that prepares the MFMA operands costs more than the vector sums:
// a two-token pass of two 1024 x 2816 layers takes 74.6 us so and 92.2 by MFMA, of the 256 x 688 decoder
// 58.8 and 70.4; of 2048-wide layers, whose products are larger, the MFMA kernels take less.
bool linear_pair_ok(int K, int N) { return K <= kPairMaxK && (size_t)K * N <= (size_t)2 << 20; }

hipError_t launch_linear_pair(const float* x, int K, float eps, const uint16_t* Wq, int Nq, const uint16_t* Wk,
                              const uint16_t* Wv, int Nkv, const float* resid, float* yq, uint16_t* yk,
                              uint16_t* yv, hipStream_t s) {
  if ((K & 7) != 0 || !linear_pair_ok(K, Nq + 2 * Nkv) || Nq < 1 || Nkv < 0) return hipErrorInvalidValue;
  ProfScope prof("linear_pair", s);
  klaunch(linear_pair_kernel, ceil_div(Nq + 2 * Nkv, kLinWaves), kLinThreads, 0, s, x, K, eps,
          reinterpret_cast<const uint4*>(Wq), Nq, reinterpret_cast<const uint4*>(Wk),
          reinterpret_cast<const uint4*>(Wv), Nkv, resid, yq, yk, yv);
  return hipGetLastError();
}

hipError_t launch_draft_tail(const float* logits, int V, int32_t* seq, int slot,
                             int32_t* cache_pos, int pos_delta, int32_t* trace_drafted,
                             hipStream_t s) {
  ProfScope prof("draft_tail", s);
  klaunch(draft_tail_kernel, 1, kTailThreads, 0, s, logits, V, seq, slot, cache_pos, pos_delta,
          trace_drafted);
  return hipGetLastError();
}

hipError_t launch_period_tail(int32_t* seq, int n, const int32_t* accept_len,
                              const int32_t* next_token, int32_t* cache_pos, int32_t* out,
                              int32_t* out_count, int out_cap, int32_t* tr_accept,
                              int32_t* tr_next, hipStream_t s) {
  ProfScope prof("period_tail", s);
  klaunch(period_tail_kernel, 1, 64, 0, s, seq, n, accept_len, next_token, cache_pos, out,
          out_count, out_cap, tr_accept, tr_next);
  return hipGetLastError();
}

}  // namespace sirius
