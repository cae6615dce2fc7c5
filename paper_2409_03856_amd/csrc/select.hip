// Radix select of the k-th largest magnitude of n fp32 values on gfx950.
//
// Non-negative IEEE floats order like their bit patterns, so the k-th largest is found digit by
// digit, most significant first (bits 30-20, 19-9, 8-0): a grid-wide histogram of the current
// digit over the values that match the digits already fixed (LDS histograms merged with integer
// atomics, so the counts are exact), whose k-th largest digit every workgroup of the next pass
// finds for itself from the merged counts. Three passes and a last one-workgroup pick give the
// exact value: four launches, three reads of the values (from the last-level cache after the
// first), bound by LDS and global atomics and by launches. For 256 x 14336 values the kernels take
// 25 us in all (8.1, 7.3, 5.0 and 4.6; four passes of 8 bits with one-thread picks between them, nine
// launches: 86). Used by the threshold calibration.
#include "common.h"
#include "kernels.h"
#include "profile.h"

namespace sirius {
namespace {

constexpr int kBins = 2048;          // 11-bit digits
constexpr int kPasses = 3;
constexpr int kSelThreads = 1024;
constexpr int kSelWaves = kSelThreads / kWave;
constexpr int kCopies = 4;           // LDS histograms: hot bins spread over them by lane
constexpr int kSelBlocks = 128;      // each merges its bins with global atomics: with 512 of half the
                                     // size the select took half as long again

struct SelectState {
  uint32_t prefix;  // bits fixed so far
  int rem;          // rank still to find among the matching values
};

__host__ __device__ constexpr int shift_of(int pass) { return pass == 0 ? 20 : (pass == 1 ? 9 : 0); }
__host__ __device__ constexpr int bins_of(int pass) { return pass == 2 ? 512 : kBins; }

// The digit of the rem-th largest value in the merged histogram gh (bins in ascending digit order),
// and the rank left inside it. Every thread of the workgroup returns both.
__device__ void pick(const int* __restrict__ gh, int bins, int rem, int* digit, int* left) {
  constexpr int kPer = kBins / kSelThreads;
  __shared__ int s_w[kSelWaves], s_out[2];
  const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid >> 6;
  // thread t holds the kPer bins below top - kPer t, in descending order
  int c[kPer], sum = 0;
#pragma unroll
  for (int i = 0; i < kPer; ++i) {
    const int b = bins - 1 - (kPer * tid + i);
    c[i] = b >= 0 ? gh[b] : 0;
    sum += c[i];
  }
  int incl = sum;
#pragma unroll
  for (int o = 1; o < kWave; o <<= 1) {
    const int t = __shfl_up(incl, o, kWave);
    if (lane >= o) incl += t;
  }
  __syncthreads();  // an earlier pick's readers are done
  if (lane == kWave - 1) s_w[wave] = incl;
  __syncthreads();
  int before = incl - sum;
  for (int w = 0; w < wave; ++w) before += s_w[w];
  if (before < rem && before + sum >= rem) {  // exactly one thread: the counts add up to >= rem
    int r = rem - before, at = -1;
#pragma unroll
    for (int i = 0; i < kPer; ++i) {
      if (at < 0) {
        if (c[i] >= r) at = i;
        else r -= c[i];
      }
    }
    s_out[0] = bins - 1 - (kPer * tid + at);
    s_out[1] = r;
  }
  __syncthreads();
  *digit = s_out[0];
  *left = s_out[1];
}

// state[p] (p > 0): the prefix and rank going into pass p, from state[p - 1] and pass p - 1's counts.
__device__ __forceinline__ SelectState state_of(int pass, int k, const SelectState* st, const int* ghist) {
  SelectState s = pass <= 1 ? SelectState{0u, k} : st[pass - 1];
  if (pass > 0) {
    int dg, left;
    pick(ghist + (pass - 1) * kBins, bins_of(pass - 1), s.rem, &dg, &left);
    s.prefix |= (uint32_t)dg << shift_of(pass - 1);
    s.rem = left;
  }
  return s;
}

__global__ __launch_bounds__(kSelThreads) void select_clear_kernel(int* __restrict__ ghist) {
  for (int i = threadIdx.x; i < kPasses * kBins; i += kSelThreads) ghist[i] = 0;
}

template <int PASS>
__global__ __launch_bounds__(kSelThreads) void select_hist_kernel(const float* __restrict__ v, int n,
                                                                  int k, SelectState* st, int* ghist) {
  constexpr int kShift = shift_of(PASS), kNb = bins_of(PASS);
  constexpr int kAhead = 4;  // float4 loads in flight per thread
  __shared__ int h[kCopies * kNb];
  const int tid = threadIdx.x;
  for (int i = tid; i < kCopies * kNb; i += kSelThreads) h[i] = 0;
  const SelectState s = state_of(PASS, k, st, ghist);
  if (PASS > 0 && blockIdx.x == 0 && tid == 0) st[PASS] = s;
  __syncthreads();
  const uint32_t fixed = PASS == 0 ? 0u : s.prefix >> shift_of(PASS > 0 ? PASS - 1 : 0);
  int* hc = h + (tid & (kCopies - 1)) * kNb;
  auto count = [&](float f) {
    const uint32_t u = __float_as_uint(f) & 0x7fffffffu;
    if (PASS == 0 || (u >> shift_of(PASS > 0 ? PASS - 1 : 0)) == fixed)
      atomicAdd(&hc[(u >> kShift) & (kNb - 1)], 1);
  };
  const int n4 = n >> 2, stride = gridDim.x * kSelThreads;
  const float4* v4 = reinterpret_cast<const float4*>(v);
  for (int i0 = blockIdx.x * kSelThreads + tid; i0 < n4; i0 += kAhead * stride) {
    float4 f[kAhead];
#pragma unroll
    for (int u = 0; u < kAhead; ++u)
      if (i0 + u * stride < n4) f[u] = v4[i0 + u * stride];
#pragma unroll
    for (int u = 0; u < kAhead; ++u)
      if (i0 + u * stride < n4) {
        count(f[u].x);
        count(f[u].y);
        count(f[u].z);
        count(f[u].w);
      }
  }
  if (blockIdx.x == 0 && tid < (n & 3)) count(v[4 * n4 + tid]);
  __syncthreads();
  for (int b = tid; b < kNb; b += kSelThreads) {
    int c = 0;
#pragma unroll
    for (int u = 0; u < kCopies; ++u) c += h[u * kNb + b];
    if (c != 0) atomicAdd(&ghist[PASS * kBins + b], c);
  }
}

__global__ __launch_bounds__(kSelThreads) void select_pick_kernel(int k, const SelectState* st,
                                                                  const int* ghist, float* out_value) {
  const SelectState s = state_of(kPasses, k, st, ghist);
  if (threadIdx.x == 0) out_value[0] = __uint_as_float(s.prefix);
}

}  // namespace

size_t select_ws_bytes() { return 256 + kPasses * kBins * sizeof(int); }

int* select_zero_ints(char* ws, int* count) {
  *count = kPasses * kBins;
  return reinterpret_cast<int*>(ws + 256);
}

hipError_t launch_select_clear(char* ws, hipStream_t stream) {
  ProfScope prof("select_clear", stream);
  klaunch(select_clear_kernel, 1, kSelThreads, 0, stream, reinterpret_cast<int*>(ws + 256));
  return hipGetLastError();
}

hipError_t launch_select_kth_largest(const float* v, int n, int k, float* out_value, char* ws,
                                     hipStream_t stream) {
  SelectState* st = reinterpret_cast<SelectState*>(ws);
  int* ghist = reinterpret_cast<int*>(ws + 256);
  const int blocks = std::max(1, std::min(kSelBlocks, ceil_div(n, kSelThreads * 16)));
  {
    ProfScope prof("select_hist", stream);
    klaunch(select_hist_kernel<0>, blocks, kSelThreads, 0, stream, v, n, k, st, ghist);
    klaunch(select_hist_kernel<1>, blocks, kSelThreads, 0, stream, v, n, k, st, ghist);
    klaunch(select_hist_kernel<2>, blocks, kSelThreads, 0, stream, v, n, k, st, ghist);
  }
  ProfScope prof("select_pick", stream);
  klaunch(select_pick_kernel, 1, kSelThreads, 0, stream, k, st, ghist, out_value);
  return hipGetLastError();
}

}  // namespace sirius
