// Gate activations of a calibration set on MFMA (gfx950): |SiLU(x_n . W_gate[i])| for N inputs and
// every neuron, into act [N][F] (the threshold is a rank of them, select.hip).
//
// The inputs stay fp32: x is split into three bf16 pieces (hi + mid + lo = x exactly), and the
// products of the pieces, exact in fp32, add up in one accumulator, so a product costs three
// bf16 MFMAs and the work is a [N x 3d] by [3d x F] matrix product: 90 GFLOP for 256 inputs of a
// 4096 x 14336 gate, bound by the MFMA rate (75 us at the 1.21 PFLOP/s of a large library product;
// 95-100 here, the matrix units busy for half of the cycles) and by the LDS reads that feed it (16
// rows of each operand per 16 x 16 x 32 product), not by HBM.
//
// Calls of a few inputs take the vector kernel of the top-k gate pass (ffn_gemv.hip) instead.
//
//  calib_gate_kernel   64 inputs x 128 neurons per workgroup, two workgroups per CU. K moves in
//                      stages of 64 columns (whole 128-byte lines) by direct global-to-LDS loads
//                      into two slots, the next stage in flight while one is multiplied; a wave
//                      forms 32 inputs x 64 neurons, so an LDS read feeds 2.4 MFMAs. The
//                      workgroups of one neuron tile run on one XCD, so its weights come from HBM
//                      once.
#include "common.h"
#include "kernels.h"
#include "profile.h"
#include "ring.h"

namespace sirius {
namespace {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8_t;
typedef __attribute__((__vector_size__(4 * sizeof(float)))) float floatx4_t;

constexpr int kThreads = 256;
constexpr int kTok = 64, kNeu = 128, kPieces = 3;
constexpr int kRows = kNeu + kPieces * kTok;   // LDS rows of a stage
constexpr int kKS = 64;                        // columns per stage
constexpr int kCpr = kKS / 8;                  // 16-byte chunks per row
constexpr int kSlot = kRows * kKS * 2;         // 40 KiB
constexpr int kLoads = kRows * kCpr / kThreads;
constexpr int kXcd = 8;
static_assert(kRows * kCpr % kThreads == 0, "whole loads");

__device__ __align__(16) uint4 g_zero_chunk[1] = {{0u, 0u, 0u, 0u}};  // source of a K tail

__device__ __forceinline__ int swz(int r, int c) { return c ^ (r & 7); }

// The product of an input with a weight row, from the input's pieces (`step` apart) put together
// again; every lane of the wave returns it.
__device__ __noinline__ float whole_dot(const uint16_t* __restrict__ xp, size_t step, const uint16_t* __restrict__ w, int d) {
  const int lane = threadIdx.x & (kWave - 1);
  float acc = 0.f;
  for (int c = 8 * lane; c < d; c += 8 * kWave) {
    __attribute__((aligned(16))) float x[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int p = kPieces - 1; p >= 0; --p) {  // lo first: exact
      const uint4 v = *reinterpret_cast<const uint4*>(xp + p * step + c);
      const uint32_t u[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        x[2 * e] += bf16_lo(u[e]);
        x[2 * e + 1] += bf16_hi(u[e]);
      }
    }
    acc = dot8(*reinterpret_cast<const uint4*>(w + c), x, acc);
  }
  return wave_sum(acc);
}

// xp [3][npad][d]: the inputs' pieces, zero rows past nb (npad a multiple of 64). zero_ints: words
// that the first workgroup clears for the select.
__global__ __launch_bounds__(kThreads, 2) void calib_gate_kernel(
    const uint16_t* __restrict__ xp, int nb, int npad, const uint16_t* __restrict__ wg, int d, int F,
    int ntok, float* __restrict__ act, int* __restrict__ zero_ints, int nzero) {
  __shared__ __attribute__((aligned(16))) unsigned char lds[2 * kSlot];
  const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid >> 6;
  const int fr = lane & 15, grp = lane >> 4;
  if (blockIdx.x == 0)
    for (int i = tid; i < nzero; i += kThreads) zero_ints[i] = 0;
  const int slot_id = blockIdx.x / kXcd;
  const int nt = blockIdx.x % kXcd + kXcd * (slot_id / ntok), tt = slot_id % ntok;
  const int n0 = nt * kNeu, m0 = tt * kTok;
  if (n0 >= F) return;  // uniform: the grid is rounded up to whole XCD rows

  // piece q * 256 + tid of a stage is row piece / 8; it holds chunk swz(row, piece % 8)
  const uint16_t* src[kLoads];
  int kofs[kLoads];
#pragma unroll
  for (int q = 0; q < kLoads; ++q) {
    const int p = q * kThreads + tid, r = p / kCpr;
    kofs[q] = 8 * swz(r, p % kCpr);
    if (r < kNeu) {
      src[q] = wg + (size_t)min(n0 + r, F - 1) * d;  // rows past d_ff: never stored
    } else {
      const int pc = (r - kNeu) / kTok, m = (r - kNeu) % kTok;
      src[q] = xp + ((size_t)pc * npad + m0 + m) * d;
    }
  }
  const int wbase = __builtin_amdgcn_readfirstlane(wave * kWave);
  auto issue = [&](int b) {
    const int k0 = b * kKS;
    const bool tail = k0 + kKS > d;  // uniform
    unsigned char* s = lds + (b & 1) * kSlot;
#pragma unroll
    for (int q = 0; q < kLoads; ++q) {
      const void* gp = (tail && k0 + kofs[q] >= d) ? static_cast<const void*>(g_zero_chunk)
                                                   : static_cast<const void*>(src[q] + k0 + kofs[q]);
      auto* lp = reinterpret_cast<__attribute__((address_space(3))) void*>(
          reinterpret_cast<size_t>(s + (q * kThreads + wbase) * 16));  // lane l lands at + 16 l
      __builtin_amdgcn_global_load_lds(gp, lp, 16, 0, 0);
    }
  };
  const int th = wave & 1, nh = wave >> 1;
  // the mid and lo pieces' sums (2^-8 of the hi ones) in accumulators of their own, the hi ones
  // added to the total every eight K steps: against 64 bits the activations of a 4096-wide gate are
  // then 1.4e-7 off (relative 2-norm; 1.65e-7 by the vector kernels before, 3.3e-7 with the hi sums
  // in two halves of K)
  floatx4_t acc[2][4], low[2][4], sum[2][4];
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int b = 0; b < 4; ++b) acc[a][b] = low[a][b] = sum[a][b] = floatx4_t{0.f, 0.f, 0.f, 0.f};
  const int nblk = (d + kKS - 1) / kKS;
  issue(0);
  for (int b = 0; b < nblk; ++b) {
    wait_vm<0>();     // this wave's loads of stage b have landed
    ring_barrier();   // and every wave's; every wave is done reading the other slot
    if (b + 1 < nblk) issue(b + 1);
    if (b != 0 && (b & 3) == 0) {  // eight K steps of 32
#pragma unroll
      for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int n = 0; n < 4; ++n) {
          sum[a][n] += acc[a][n];
          acc[a][n] = floatx4_t{0.f, 0.f, 0.f, 0.f};
        }
    }
    const unsigned char* s = lds + (b & 1) * kSlot;
#pragma unroll
    for (int i = 0; i < kKS / 32; ++i) {
      const int c = 4 * i + grp;
      auto row = [&](int r) {
        return *reinterpret_cast<const bf16x8_t*>(s + r * (kKS * 2) + 16 * swz(r, c));
      };
      bf16x8_t bw[4], ax[kPieces][2];
#pragma unroll
      for (int n = 0; n < 4; ++n) bw[n] = row(64 * nh + 16 * n + fr);
#pragma unroll
      for (int p = 0; p < kPieces; ++p)
#pragma unroll
        for (int a = 0; a < 2; ++a) ax[p][a] = row(kNeu + p * kTok + 32 * th + 16 * a + fr);
#pragma unroll
      for (int p = 0; p < kPieces; ++p)
#pragma unroll
        for (int a = 0; a < 2; ++a)
#pragma unroll
          for (int n = 0; n < 4; ++n) {
            floatx4_t& s4 = p == 0 ? acc[a][n] : low[a][n];
            s4 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ax[p][a], bw[n], s4, 0, 0, 0);
          }
    }
  }
  // C layout: lane holds neuron fr of a tile and inputs 4 grp + e
  bool nan = false;
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int n = 0; n < 4; ++n) {
      const int j = n0 + 64 * nh + 16 * n + fr;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int m = m0 + 32 * th + 16 * a + 4 * grp + e;
        const float g = (sum[a][n][e] + acc[a][n][e]) + low[a][n][e];
        nan |= g != g;
        if (m < nb && j < F) act[(size_t)m * F + j] = fabsf(silu(g));
      }
    }
  // an infinite weight times a zero piece, or times pieces of both signs, is NaN where the product is
  // an infinity: the wave forms such values again from whole inputs
  if (__builtin_expect(__ballot(nan) == 0, 1)) return;
  for (int i = 0; i < 32; ++i) {
    const int at = m0 + 32 * th + 16 * (i >> 4) + (i & 3), n = n0 + 64 * nh + 16 * ((i >> 2) & 3);
    const bool live = at + 4 * grp < nb && n + fr < F;
    const float v = live ? act[(size_t)(at + 4 * grp) * F + n + fr] : 0.f;
    for (unsigned long long left = __ballot(v != v); left != 0; left &= left - 1) {
      const int l = __builtin_ctzll(left);
      const size_t m = at + 4 * (l >> 4), j = n + (l & 15);
      const float g = whole_dot(xp + m * d, (size_t)npad * d, wg + j * d, d);
      if (lane == l) act[m * F + j] = fabsf(silu(g));
    }
  }
}

constexpr int kChunk = 1024;  // inputs per launch: bounds the pieces' workspace

}  // namespace

size_t gate_absact_ws(int N, int d) {
  return (size_t)kPieces * std::min(kChunk, ceil_div(N, kTok) * kTok) * d * 2;
}

// At most four inputs that leave room for two workgroups' copies of them in LDS: the vector kernel
// streams the gate at HBM rate, where the MFMA kernel fills its 64-input tiles with zeros on d_ff / 128
// workgroups. The whole call for 1, 2 and 4 inputs of 4096 x 14336 34, 38 and 56 us against 77, 78 and
// 80; 2 of 8192 x 28672 104 against 176, but 3, one workgroup per CU, 195 against 173.
bool calib_few(int N, int d) { return N <= 4 && N * d <= 16384; }

hipError_t launch_gate_absact(const float* x, int N, const uint16_t* wg, int d, int F, float* act,
                              char* ws, char* sel_ws, hipStream_t stream) {
  if (calib_few(N, d)) {
    hipError_t e = launch_select_clear(sel_ws, stream);
    if (e != hipSuccess) return e;
    return launch_gate_act(x, N, wg, d, F, -1.f, act, stream, "calib_gate");
  }
  int nzero = 0;
  int* zero_ints = select_zero_ints(sel_ws, &nzero);
  uint16_t* xp = reinterpret_cast<uint16_t*>(ws);
  for (int n0 = 0; n0 < N; n0 += kChunk) {
    const int nb = std::min(kChunk, N - n0);
    const int ntok = ceil_div(nb, kTok), npad = ntok * kTok;
    {
      ProfScope prof("calib_prep", stream);
      hipError_t e = launch_prep_pieces3(x + (size_t)n0 * d, nb, d, npad, xp, stream);
      if (e != hipSuccess) return e;
    }
    ProfScope prof("calib_gate", stream);
    const int grid = kXcd * ceil_div(ceil_div(F, kNeu), kXcd) * ntok;
    klaunch(calib_gate_kernel, grid, kThreads, 0, stream, xp, nb, npad, wg, d, F, ntok,
            act + (size_t)n0 * F, zero_ints, nzero);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

}  // namespace sirius
