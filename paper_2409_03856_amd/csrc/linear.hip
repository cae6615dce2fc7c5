// Projections of a chunk of 2..64 tokens on MFMA (gfx950): y = xn W^T for up to three weight
// matrices in one launch (a layer's q, k and v, the output projection, the LM head), with the
// chunk's RMSNorm, the residual and the bf16 stores of keys and values folded in.
//
//  prep_frag_kernel        x -> optional RMSNorm -> three bf16 pieces (hi + mid + lo = x exactly,
//                          each the bf16 rounding of what the previous ones leave, so the MFMA
//                          products of the pieces sum to the fp32 product; the first alone is x
//                          rounded to bf16, the batched FFN's dense input), stored in the order
//                          in which the lanes of an MFMA take them, zero past the last token
//                          and past K.
//  linear_mfma_kernel<..>  one workgroup per 16 RT weight rows: the rows stream through LDS in
//                          blocks of KB columns (registers, two blocks ahead, then two LDS
//                          buffers: HBM wants whole runs of a row per request, an MFMA wants 16
//                          rows), wave w multiplies quarter w of every block by the x pieces,
//                          which it reads from L2 in operand order; the four partials are summed
//                          in wave order at the end.
//
// Bound: HBM and the L2 reads of the x pieces, one read of the weights per call (2 N K bytes) whatever
// the number of tokens; the products are 6 n flops per weight, 12 % of the MFMA rate at 16 tokens.
#include "common.h"
#include "kernels.h"
#include "profile.h"
#include "ring.h"

namespace sirius {
namespace {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8_t;
typedef __attribute__((__vector_size__(4 * sizeof(float)))) float floatx4_t;

constexpr int kLmThreads = 256;
constexpr int kLmWaves = kLmThreads / kWave;
constexpr int kPieces = 3;

// x pieces: [K step of 32][piece][16-token tile][lane][8 values]; lane = 16 (k % 32 / 8) + m % 16.
// One workgroup per padded token row, which passes through LDS. The RMSNorm sums are those of
// rmsnorm_vec_kernel (thread t of 256 takes float4s t + 256 u in ascending order, the wave sums in
// wave order), so the normalised row is bit for bit that kernel's; then each thread forms the pieces
// of one operand chunk of eight values. Bound by latency: 1024 threads, of which the first 256 form
// the sums, take 4.1-5.0 us at 4096 columns and 6.0 at 8192 (256 threads: 5.5 and 8.2-9.5).
constexpr int kPrepThreads = 1024;
__global__ __launch_bounds__(kPrepThreads) void prep_frag_kernel(const float* __restrict__ x, int n, int K,
                                                                 int ksteps, float norm_eps, int MT,
                                                                 int pieces, uint4* __restrict__ xf) {
  __shared__ float s_w[4];
  __shared__ float4 s_x[2048];
  const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid >> 6;
  const int m = blockIdx.x, mt = m >> 4;
  const int k4 = K >> 2, k8 = K >> 3;
  float inv = 1.f;
  if (m < n) {  // uniform over the workgroup
    const float4* xr = reinterpret_cast<const float4*>(x + (size_t)m * K);
#pragma unroll
    for (int u = 0; u < 2; ++u) {  // K <= 8192
      const int e = tid + kPrepThreads * u;
      if (e < k4) s_x[e] = xr[e];
    }
    __syncthreads();
    if (norm_eps >= 0.f) {
      if (wave < 4) {
        float ss = 0.f;
#pragma unroll
        for (int u = 0; u < 8; ++u) {
          const int e = tid + 256 * u;
          const float4 v = (e < k4) ? s_x[e] : make_float4(0.f, 0.f, 0.f, 0.f);
          ss = fmaf(v.x, v.x, ss);
          ss = fmaf(v.y, v.y, ss);
          ss = fmaf(v.z, v.z, ss);
          ss = fmaf(v.w, v.w, ss);
        }
        ss = wave_sum(ss);
        if (lane == 0) s_w[wave] = ss;
      }
      __syncthreads();
      const float tot = ((s_w[0] + s_w[1]) + s_w[2]) + s_w[3];
      inv = 1.0f / sqrtf(tot / (float)K + norm_eps);
    }
  }
  for (int c = tid; c < 4 * ksteps; c += kPrepThreads) {  // operand chunk c: values 8 c .. 8 c + 7
    float r[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    if (m < n && c < k8) {
      const float4 a = s_x[2 * c], b = s_x[2 * c + 1];
      r[0] = a.x * inv; r[1] = a.y * inv; r[2] = a.z * inv; r[3] = a.w * inv;
      r[4] = b.x * inv; r[5] = b.y * inv; r[6] = b.z * inv; r[7] = b.w * inv;
    }
    bool top = false;
#pragma unroll
    for (int e = 0; e < 8; ++e) top |= rounds_to_inf(r[e]);
    auto write = [&](auto piece_of) {
#pragma unroll
      for (int p = 0; p < kPieces; ++p) {
        if (p == pieces) break;  // uniform
        uint32_t b[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) b[e] = piece_of(r[e]);
        xf[(((size_t)(c >> 2) * pieces + p) * MT + mt) * kWave + 16 * (c & 3) + (m & 15)] =
            make_uint4(b[0] | (b[1] << 16), b[2] | (b[3] << 16), b[4] | (b[5] << 16),
                       b[6] | (b[7] << 16));
      }
    };
    if (pieces > 1 && __builtin_expect(top, 0)) write(take_piece_any);
    else write(take_piece);  // a single piece is the rounding, also to an infinity
  }
}

struct LinearOut {
  const uint16_t *Wq, *Wk, *Wv;  // rows [0, Nq) of Wq, then Nkv rows of Wk, Nkv of Wv
  const float* resid;            // added to yq, or null
  float* yq;                     // [n][Nq]
  uint16_t *yk, *yv;             // [n][Nkv] bf16
  int Nq, Nkv;
};

// Row j of the launch's weight rows.
__device__ __forceinline__ const uint4* row_of(const LinearOut& o, int j, int K) {
  const uint16_t* w = j < o.Nq ? o.Wq + (size_t)j * K
                      : j < o.Nq + o.Nkv ? o.Wk + (size_t)(j - o.Nq) * K
                                         : o.Wv + (size_t)(j - o.Nq - o.Nkv) * K;
  return reinterpret_cast<const uint4*>(w);
}

// The product of token m's row with a weight row as linear_kernel (model.hip) forms it, from the x
// pieces put together again; every lane of the wave returns it.
template <int MT>
__device__ __noinline__ float whole_dot(const uint4* __restrict__ xf, int m, const uint4* __restrict__ w, int K) {
  const int lane = threadIdx.x & (kWave - 1);
  float acc = 0.f;
  for (int c = lane; c < K >> 3; c += kWave) {
    __attribute__((aligned(16))) float x[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int p = kPieces - 1; p >= 0; --p) {  // lo first: exact
      const uint4 v = xf[(((size_t)(c >> 2) * kPieces + p) * MT + (m >> 4)) * kWave + 16 * (c & 3) + (m & 15)];
      const uint32_t u[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        x[2 * e] += bf16_lo(u[e]);
        x[2 * e + 1] += bf16_hi(u[e]);
      }
    }
    acc = dot8(w[c], x, acc);
  }
  return wave_sum(acc);
}

// MT 16-token tiles, RT 16-row weight tiles per workgroup, KB columns per block, D blocks in flight.
template <int MT, int RT, int KB, int D>
__global__ __launch_bounds__(kLmThreads) void linear_mfma_kernel(const uint4* __restrict__ xf,
                                                                 int n, int K, int ksteps,
                                                                 LinearOut o) {
  constexpr int kRows = 16 * RT;
  constexpr int kCpr = KB / 8;                        // 16-byte chunks per row and block
  constexpr int kLd = kRows * kCpr / kLmThreads;      // loads per thread and block
  constexpr int kRowStep = kLmThreads / kCpr;         // rows between a thread's loads
  constexpr int kPitch = KB * 2 + 16;                 // the 16 rows of an operand read: all banks
  constexpr int kBuf = kRows * kPitch;
  constexpr int kSteps = KB / 32 / kLmWaves;          // K steps per wave and block
  static_assert(kRows * kCpr % kLmThreads == 0 && kLmThreads % kCpr == 0, "whole loads");
  constexpr int kRed = kLmWaves * RT * MT * kWave * 16;
  __shared__ __attribute__((aligned(16))) unsigned char lds[2 * kBuf > kRed ? 2 * kBuf : kRed];
  const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid >> 6;
  const int fr = lane & 15, grp = lane >> 4;
  const int N = o.Nq + 2 * o.Nkv, n0 = blockIdx.x * kRows;
  const int k8 = K >> 3, nblk = (K + KB - 1) / KB;

  const int ch = tid % kCpr, row0 = tid / kCpr;
  const uint4* src[kLd];
#pragma unroll
  for (int i = 0; i < kLd; ++i) {
    const int j = min(n0 + row0 + i * kRowStep, N - 1);  // rows past the last: never stored
    src[i] = row_of(o, j, K) + ch;
  }
  static_assert(D % 2 == 0, "LDS and x buffers alternate");
  uint4 wr[D][kLd];
  auto load_w = [&](uint4(&r)[kLd], int b) {
    const bool ok = b * kCpr + ch < k8;
#pragma unroll
    for (int i = 0; i < kLd; ++i) r[i] = ok ? ld_stream(src[i] + b * kCpr) : make_uint4(0u, 0u, 0u, 0u);
  };
  auto store_w = [&](const uint4(&r)[kLd], int buf) {
#pragma unroll
    for (int i = 0; i < kLd; ++i)
      *reinterpret_cast<uint4*>(lds + buf * kBuf + (row0 + i * kRowStep) * kPitch + 16 * ch) = r[i];
  };
  // x pieces of this wave's K steps of block b (zero past the padded K)
  uint4 xa[2][kSteps][kPieces][MT];
  auto load_x = [&](uint4(&r)[kSteps][kPieces][MT], int b) {
#pragma unroll
    for (int i = 0; i < kSteps; ++i) {
      const int st = b * (KB / 32) + kSteps * wave + i;
#pragma unroll
      for (int p = 0; p < kPieces; ++p)
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
          r[i][p][mt] = st < ksteps ? xf[(((size_t)st * kPieces + p) * MT + mt) * kWave + lane]
                                    : make_uint4(0u, 0u, 0u, 0u);
    }
  };
  // a block's products are summed from zero, the hi pieces apart from the rest, and then added to
  // the total: the logits of an 8192-wide pass are then 4.0e-7 off 64 bits (5.8e-7 with one chain
  // of products over all of K, 4.5e-7 by the vector kernels before)
  floatx4_t acc[RT][MT];
#pragma unroll
  for (int rt = 0; rt < RT; ++rt)
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) acc[rt][mt] = floatx4_t{0.f, 0.f, 0.f, 0.f};
  auto step = [&](uint4(&wcur)[kLd], uint4(&xcur)[kSteps][kPieces][MT],
                  uint4(&xnext)[kSteps][kPieces][MT], int b) {
    store_w(wcur, b & 1);
    if (b + D < nblk) load_w(wcur, b + D);
    if (b + 1 < nblk) load_x(xnext, b + 1);
    ring_barrier();  // block b is in its buffer; every wave is done with block b - 1's reads
    const unsigned char* buf = lds + (b & 1) * kBuf;
    bf16x8_t bw[kSteps][RT];
#pragma unroll
    for (int i = 0; i < kSteps; ++i)
#pragma unroll
      for (int rt = 0; rt < RT; ++rt)
        bw[i][rt] = *reinterpret_cast<const bf16x8_t*>(buf + (16 * rt + fr) * kPitch +
                                                       64 * (kSteps * wave + i) + 16 * grp);
#pragma unroll
    for (int rt = 0; rt < RT; ++rt)
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) {
        floatx4_t sh = floatx4_t{0.f, 0.f, 0.f, 0.f}, sl = sh;
#pragma unroll
        for (int p = 2; p > 0; --p)
#pragma unroll
          for (int i = 0; i < kSteps; ++i)
            sl = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, xcur[i][p][mt]),
                                                         bw[i][rt], sl, 0, 0, 0);
#pragma unroll
        for (int i = 0; i < kSteps; ++i)
          sh = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, xcur[i][0][mt]),
                                                       bw[i][rt], sh, 0, 0, 0);
        acc[rt][mt] += sh + sl;
      }
  };
#pragma unroll
  for (int u = 0; u < D; ++u)
    if (u < nblk) load_w(wr[u], u);
  load_x(xa[0], 0);
  for (int b = 0; b < nblk; b += D) {
#pragma unroll
    for (int u = 0; u < D; ++u)
      if (b + u < nblk) step(wr[u], xa[u & 1], xa[1 - (u & 1)], b + u);
  }

  // the four waves' sums in wave order; C layout: lane l holds weight row l & 15 of the tile and
  // tokens 4 (l >> 4) + e
  __syncthreads();
  floatx4_t* red = reinterpret_cast<floatx4_t*>(lds);
#pragma unroll
  for (int rt = 0; rt < RT; ++rt)
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) red[((wave * RT + rt) * MT + mt) * kWave + lane] = acc[rt][mt];
  __syncthreads();
  const float* rf = reinterpret_cast<const float*>(lds);
  auto sum_of = [&](int jr, int m) {
    const int at = (((jr >> 4) * MT + (m >> 4)) * kWave + 16 * ((m & 15) >> 2) + (jr & 15)) * 4 + (m & 3);
    float s = rf[at];
#pragma unroll
    for (int w = 1; w < kLmWaves; ++w) s += rf[at + w * RT * MT * kWave * 4];
    return s;
  };
  auto store = [&](int j, int m, float s) {
    if (j < o.Nq) {
      const size_t e = (size_t)m * o.Nq + j;
      o.yq[e] = o.resid != nullptr ? o.resid[e] + s : s;
    } else if (j < o.Nq + o.Nkv) {
      o.yk[(size_t)m * o.Nkv + j - o.Nq] = (uint16_t)f32_to_bf16(s);
    } else {
      o.yv[(size_t)m * o.Nkv + j - o.Nq - o.Nkv] = (uint16_t)f32_to_bf16(s);
    }
  };
  bool nan = false;
  for (int i = tid; i < kRows * n; i += kLmThreads) {
    const int jr = i % kRows, m = i / kRows;
    if (n0 + jr >= N) continue;
    const float s = sum_of(jr, m);
    if (s == s) store(n0 + jr, m, s);
    else nan = true;
  }
  // an infinite weight times a zero piece, or times pieces of both signs, is NaN where the product is
  // an infinity: such sums are formed again from whole values, a wave per sum
  if (__builtin_expect(__ballot(nan) == 0, 1)) return;
  for (int i0 = tid - lane; i0 < kRows * n; i0 += kLmThreads) {
    const int i = i0 + lane, jr = i % kRows, m = i / kRows;
    const bool live = m < n && n0 + jr < N;
    const float s = live ? sum_of(jr, m) : 0.f;
    for (unsigned long long left = __ballot(s != s); left != 0; left &= left - 1) {
      const int l = __builtin_ctzll(left);
      const int jl = n0 + __shfl(jr, l, kWave), ml = __shfl(m, l, kWave);
      const float t = whole_dot<MT>(xf, ml, row_of(o, jl, K), K);
      if (lane == l) store(jl, ml, t);
    }
  }
}

}  // namespace

hipError_t launch_prep_frag(const float* x, int n, int K, float eps, int pieces, char* xf, hipStream_t s) {
  if ((K & 7) != 0 || K > 8192 || n < 1 || pieces < 1 || pieces > kPieces) return hipErrorInvalidValue;
  const int MT = ceil_div(n, 16);
  klaunch(prep_frag_kernel, 16 * MT, kPrepThreads, 0, s, x, n, K, ceil_div(K, 32), eps, MT, pieces,
          reinterpret_cast<uint4*>(xf));
  return hipGetLastError();
}

namespace {

template <int MT>
hipError_t launch_t(const float* x, int n, int K, float eps, const LinearOut& o, char* ws,
                    hipStream_t s) {
  const int ksteps = ceil_div(K, 32), N = o.Nq + 2 * o.Nkv;
  uint4* xf = reinterpret_cast<uint4*>(ws);
  {
    ProfScope prof("linear_prep", s);
    hipError_t e = launch_prep_frag(x, n, K, eps, kPieces, ws, s);
    if (e != hipSuccess) return e;
  }
  ProfScope prof("linear_mfma", s);
  // Every workgroup reads all the x pieces of its K range from L2: 3 MT / RT bytes per weight byte.
  // 64 rows per workgroup where that still gives most CUs one (LM heads): at 16 tokens and
  // 128256 x 4096 183-188 us (5.6-5.7 TB/s) against 230 with 32 rows and 250 with 16; at 32000 x 2048 27.5
  // against 41, at 24 tokens and 16000 x 4096 34 against 54. Below that 16 rows, so that a layer's
  // projections fill the chip: 6144 x 4096 and 4096 x 4096 together 31.6 us against 43 with 32 rows
  // and 47 with 64; there one 16-token tile takes 1 KiB of a row per load and four blocks in flight
  // (35 us with 512 bytes and two), unless K is too short to give every wave its part of a block.
  constexpr int kWide = 64 * 192;
  if (N >= kWide)
    klaunch(linear_mfma_kernel<MT, 4, 256, 2>, ceil_div(N, 64), kLmThreads, 0, s, xf, n, K, ksteps, o);
  else if (MT == 1 && K >= 1024)
    klaunch(linear_mfma_kernel<MT, 1, MT == 1 ? 512 : 256, MT == 1 ? 4 : 2>, ceil_div(N, 16), kLmThreads, 0,
            s, xf, n, K, ksteps, o);
  else
    klaunch(linear_mfma_kernel<MT, 1, 256, 2>, ceil_div(N, 16), kLmThreads, 0, s, xf, n, K, ksteps, o);
  return hipGetLastError();
}

}  // namespace

size_t linear_mfma_ws(int n, int K) {
  return (size_t)ceil_div(K, 32) * kPieces * ceil_div(n, 16) * kWave * 16;
}

hipError_t launch_linear_mfma(const float* x, int n, int K, float eps, const uint16_t* Wq, int Nq,
                              const uint16_t* Wk, const uint16_t* Wv, int Nkv, const float* resid,
                              float* yq, uint16_t* yk, uint16_t* yv, char* ws, hipStream_t s) {
  if ((K & 7) != 0 || K > 8192 || n < 1 || n > 64 || Nq < 1 || Nkv < 0) return hipErrorInvalidValue;
  const LinearOut o{Wq, Wk, Wv, resid, yq, yk, yv, Nq, Nkv};
  switch (ceil_div(n, 16)) {
    case 1: return launch_t<1>(x, n, K, eps, o, ws, s);
    case 2: return launch_t<2>(x, n, K, eps, o, ws, s);
    case 3: return launch_t<3>(x, n, K, eps, o, ws, s);
    default: return launch_t<4>(x, n, K, eps, o, ws, s);
  }
}

}  // namespace sirius
