// Multi-token SwiGLU FFN on MFMA (gfx950) for 2..64 tokens with d_model % 256 == 0: dense and
// condensed decode of small batches, the full model's parallel pass over a drafted chunk or tree,
// and per-token threshold (CATS) and top-k sparsity of batched tokens. The weights are streamed
// once per call whatever the batch (up to four 16-token MFMA tiles share every weight byte), so
// the call stays HBM-bound: at 16 tokens the products are 2 flops per weight byte per token,
// far below the bf16 MFMA ridge (about 300).
//
//  prep_pieces_kernel  x -> optional RMSNorm -> PX bf16 pieces, zero-padded to whole 16-token
//                      tiles, in rows (the unit kernels and the calibration read them so).
//                      PX = 1: x rounded to bf16 (the full model's pass). PX = 3: x = hi + mid
//                      + lo exactly (each piece the bf16 rounding of what the previous ones
//                      leave), so the MFMA products of the three pieces sum to the fp32 product:
//                      the threshold, top-k and small-batch paths keep fp32 inputs.
//  prep_frag_kernel    (linear.hip) the same pieces in the order of the MFMA operand registers.
//  gu_unit_kernel      dense: H = SiLU(X W_gate^T) * (X W_up^T) for one segment of at most 56
//                      neurons per workgroup, for 8..16 tokens with d_model a multiple of 2048:
//                      the weights move through LDS in units of 16 rows x 2048 columns, each
//                      row's 4 KiB requested by one wave with consecutive 1 KiB direct loads (the
//                      order in which HBM streams a row fastest), x held in registers.
//  gu_frag_kernel      the same for every other call: the weights go through registers into two
//                      LDS buffers, the x pieces from L2 into registers in operand order.
//  cats_frag_kernel    per-token sparsity over one segment: the gate rows alone (threshold mode
//                      and the top-k gate pass), SiLU, the per-token keep decision (|a| > t, or
//                      the top-k key against the token's cut), the union of the tokens' kept
//                      neurons compacted in ascending order with a wave ballot, then the up rows
//                      of that union only; h = a u where the token keeps the neuron, 0 elsewhere,
//                      stored per segment position. Up rows outside the union are never read.
//                      Dense and condensed calls of fewer than 8 tokens run here too, every
//                      neuron kept, so that a threshold below 0 gives the dense result bit for
//                      bit.
//  cats_unit_kernel    the modes of cats_frag_kernel for at most 4 tokens with d_model a multiple
//                      of 2048 on the unit layout: the three pieces of the four tokens are the 12
//                      rows of one MFMA operand tile, held in registers.
//  down_ring_kernel    Y_partial over one 256-column tile and one range of 64-position blocks of
//                      the segment layout: a segment's rows (dense) or its union rows (gathered
//                      by index), so W_down rows outside the union are never read.
//                      The W_down rows of a block and the hi/lo h fragments move into an LDS
//                      ring by direct loads.
//  reduce_kernel       (ffn_gemv.hip) y = resid + the partials in a fixed order; the per-token
//                      ascending kept lists from the per-segment lists.
//
// Every sum has a fixed order and no kernel uses atomics: results are bitwise reproducible.
#include "common.h"
#include "kernels.h"
#include "profile.h"
#include "ring.h"
#include "topk.h"

namespace sirius {
namespace {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8_t;
typedef __attribute__((__vector_size__(4 * sizeof(float)))) float floatx4_t;

__device__ __forceinline__ bf16x8_t as_bf16x8(uint4 v) { return __builtin_bit_cast(bf16x8_t, v); }

constexpr int kBT = 512;                 // threads per workgroup: eight waves
constexpr int kSegN = 56;                // neurons per segment at most
constexpr int kSegPad = 64;              // segment positions (whole 16-neuron tiles, one down block)
constexpr int kLdsRing = 150 * 1024;     // LDS the rings may take
constexpr int kDnCols = 256;             // output columns per down workgroup
constexpr int kDnBlock = 64;             // rows per down block

// vmcnt wait until at most `later` (0, 1 or 2) blocks of L loads each are still in flight
template <int L>
__device__ __forceinline__ void wait_later(int later) {
  static_assert(2 * L <= 63, "vmcnt counts up to 63 loads");
  switch (later) {
    case 0: wait_vm<0>(); break;
    case 1: wait_vm<L>(); break;
    default: wait_vm<2 * L>(); break;
  }
}

// ---- x -> optional RMSNorm -> PX bf16 pieces [PX][Mpad][d]; one workgroup per padded row.
template <int PX>
__global__ __launch_bounds__(256) void prep_pieces_kernel(const float* __restrict__ x, int B, int d,
                                                          int mpad, float norm_eps,
                                                          uint16_t* __restrict__ xp) {
  constexpr int kPer = 8;  // d_model <= 8192: 2048 float4 per row over 256 threads
  __shared__ float s_w[4];
  const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid >> 6;
  const int m = blockIdx.x;
  const int nv4 = d >> 2;
  if (m >= B) {  // uniform over the block: padded rows are zero in every piece
#pragma unroll
    for (int p = 0; p < PX; ++p) {
      uint2* out = reinterpret_cast<uint2*>(xp + ((size_t)p * mpad + m) * d);
      for (int i = tid; i < nv4; i += 256) out[i] = make_uint2(0u, 0u);
    }
    return;
  }
  const float4* xr = reinterpret_cast<const float4*>(x + (size_t)m * d);
  float4 v[kPer];
#pragma unroll
  for (int u = 0; u < kPer; ++u) {
    const int i = tid + 256 * u;
    v[u] = (i < nv4) ? xr[i] : make_float4(0.f, 0.f, 0.f, 0.f);
  }
  if (norm_eps >= 0.f) {
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
    const float inv = 1.0f / sqrtf(tot / (float)d + norm_eps);
#pragma unroll
    for (int u = 0; u < kPer; ++u) {
      v[u].x *= inv;
      v[u].y *= inv;
      v[u].z *= inv;
      v[u].w *= inv;
    }
  }
  bool top = false;
#pragma unroll
  for (int u = 0; u < kPer; ++u)
    top |= rounds_to_inf(v[u].x) || rounds_to_inf(v[u].y) || rounds_to_inf(v[u].z) || rounds_to_inf(v[u].w);
  auto write = [&](auto piece_of) {
#pragma unroll
    for (int u = 0; u < kPer; ++u) {
      const int i = tid + 256 * u;
      if (i >= nv4) continue;
      float r[4] = {v[u].x, v[u].y, v[u].z, v[u].w};
#pragma unroll
      for (int p = 0; p < PX; ++p) {
        uint32_t b[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) b[e] = piece_of(r[e]);
        reinterpret_cast<uint2*>(xp + ((size_t)p * mpad + m) * d)[i] =
            make_uint2(b[0] | (b[1] << 16), b[2] | (b[3] << 16));
      }
    }
  };
  if (PX > 1 && __builtin_expect(top, 0)) write(take_piece_any);
  else write(take_piece);
}

// Segment geometry: nseg segments of np neurons over n_rows rows, np a multiple of 4 of at most
// 56, small enough that there are at least 256 segments (one workgroup per CU) when n_rows allows.
// Above 256 full segments the rows are split over whole rounds of 256 workgroups: 15104 rows are
// 472 segments of 32 and not 270 of 56, whose second round was nearly empty (gate/up at 3 tokens
// of 4608 columns 97 -> 55 us with the operand-order pipeline, 40 tokens 196 -> 105).
struct Seg {
  int nseg, np;
};
constexpr int kSegTarget = 256;
__host__ __device__ inline Seg seg_of(int n_rows, int most) {  // segments of at most `most` neurons
  const int rounds = (n_rows + kSegTarget * most - 1) / (kSegTarget * most);
  int np = (n_rows + kSegTarget * rounds - 1) / (kSegTarget * rounds);
  np = (np + 3) & ~3;
  if (np > most) np = most;
  if (np < 4) np = 4;
  return Seg{(n_rows + np - 1) / np, np};
}
// Positions a segment owns in h and the down blocks: whole 16-neuron tiles. 48 next to 32 and 64:
// the down pass streams a row for every position (8192 columns, 22671 rows in segments of 48, 40 tokens:
// 92 us with 64 positions, 80 with 48).
__host__ __device__ constexpr int seg_positions(int np) { return np <= 16 ? 16 : (np <= 32 ? 32 : (np <= 48 ? 48 : kSegPad)); }

// h = SiLU(g) u as a bf16 pair (hi, lo): hi = bf16(h), lo = bf16(h - hi)
__device__ __forceinline__ void store_h(uint16_t* hhi, uint16_t* hlo, size_t at, float h) {
  const uint32_t hi = f32_to_bf16(h);
  const float lo = h - __uint_as_float(hi << 16);
  hhi[at] = (uint16_t)hi;
  hlo[at] = (uint16_t)f32_to_bf16(lo);
}

// h positions [npos, hs) of every token row lie past the last segment but inside the last down
// block; the last workgroup of a gate/up launch writes zeros there (hs - npos < 64)
__device__ __forceinline__ void zero_h_tail(uint16_t* hhi, uint16_t* hlo, int hs, int npos,
                                            int mpad) {
  const int tail = hs - npos;
  for (int i = threadIdx.x; i < mpad * tail; i += blockDim.x) {
    const size_t at = (size_t)(i / tail) * hs + npos + i % tail;
    hhi[at] = 0;
    hlo[at] = 0;
  }
}

// ---- dense gate/up of 8..16 tokens on the bf16-rounded input with d_model a multiple of 2048.
// HBM streams a weight row fastest when its bytes are requested close together in time: one wave
// reading a row's aligned 4 KiB with consecutive 1 KiB loads moves about 6.8 TB/s over the chip,
// the same bytes requested 256 or 512 bytes per row per instruction, or spread over later
// instructions, 5.0-6.0. This kernel
// moves the weights through LDS in units of 16 rows x 2048 columns, wave w requesting row w of
// the unit with four consecutive 1 KiB direct loads, two unit buffers (128.5 KiB of LDS).
// Segment rows: gate rows [0, np), up rows [np, 2 np), padded to whole 16-row tiles with zero
// rows; units go tile by tile with the K spans inner, so a row's spans are requested in
// consecutive units. Wave w multiplies K steps 4 w .. 4 w + 3 of every unit (x in registers for
// the whole call, the weights from LDS) into one partial per tile; the 16 partials are summed in
// wave order at the end, so the result does not depend on timing.
constexpr int kUnitThreads = 1024;                  // 16 waves: one row of a unit each
constexpr int kUnitWaves = kUnitThreads / kWave;
constexpr int kUnitK = 2048;                        // columns per unit (4 KiB of a row)
constexpr int kUnitRowBytes = kUnitK * 2 + 16;      // LDS row stride: the 16 rows of an MFMA
                                                    // operand read lie in distinct banks
constexpr int kUnitBytes = 16 * kUnitRowBytes;      // 65792
constexpr int kUnitLds = 2 * kUnitBytes;            // 131584
constexpr int kUnitTiles = (2 * kSegN + 15) / 16;   // 16-row tiles per segment at most (7)
constexpr int kUnitLoads = kUnitK * 2 / 1024;       // 1 KiB loads per wave per unit (4)
constexpr int kUnitSteps = kUnitK / 32 / kUnitWaves;  // 32-wide K steps per wave per unit (4)
static_assert(kUnitWaves * kUnitTiles * kWave * 16 + kUnitTiles * 16 * 16 * 4 <= kUnitLds,
              "the end-of-call reduction fits in the unit buffers");
__device__ __align__(16) uint16_t g_zero_row[kUnitK];  // source of the padding rows

// x operand (A) of this wave's K steps in every span: row fr of the tile from `row` (16 rows of
// d columns), zero where `ok` is false (the load is issued anyway, from row 0, so every wave's
// load count is the same)
template <int NSPAN>
__device__ __forceinline__ void unit_x(bf16x8_t (&xa)[NSPAN][kUnitSteps], const uint16_t* row,
                                       bool ok) {
  const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x >> 6, grp = lane >> 4;
#pragma unroll
  for (int s = 0; s < NSPAN; ++s)
#pragma unroll
    for (int j = 0; j < kUnitSteps; ++j) {
      uint4 v = *reinterpret_cast<const uint4*>(row + s * kUnitK + 32 * (kUnitSteps * wave + j) + 8 * grp);
      if (!ok) v = make_uint4(0u, 0u, 0u, 0u);
      xa[s][j] = as_bf16x8(v);
    }
}

// The unit pipeline: T (<= TMAX) tiles of 16 rows, row r of the sequence from row_of(r) (wave-
// uniform; nullptr: a zero row), units (tile u / NSPAN, span u % NSPAN) in two LDS buffers, wave w
// requesting row w of every unit; acc[t] = this wave's K steps of tile t. Then the waves'
// partials are summed in wave order into res[16 t + row][x row] (fp32, in LDS past the partials),
// and the unit buffers are free again. A row's result does not depend on its place in the
// sequence: the same loads, steps and sums give it wherever it sits.
template <int NSPAN, int TMAX, class RowOf>
__device__ __forceinline__ float* unit_pass(unsigned char* lds_u, int T, RowOf row_of,
                                            const bf16x8_t (&xa)[NSPAN][kUnitSteps]) {
  const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid >> 6;
  const int fr = lane & 15, grp = lane >> 4;
  const int U = T * NSPAN;
  auto issue = [&](int u) {
    const int t = u / NSPAN, sp_ = u - t * NSPAN;
    const uint16_t* row = row_of(__builtin_amdgcn_readfirstlane(16 * t + wave));  // wave-uniform
    const uint16_t* src = row != nullptr ? row + sp_ * kUnitK : g_zero_row;
    unsigned char* dst = lds_u + (u & 1) * kUnitBytes + wave * kUnitRowBytes;
#pragma unroll
    for (int q = 0; q < kUnitLoads; ++q) {
      auto* lp = reinterpret_cast<__attribute__((address_space(3))) void*>(
          reinterpret_cast<size_t>(dst + q * 1024));  // lane l lands at + 16 l
      __builtin_amdgcn_global_load_lds(src + q * 512 + 8 * lane, lp, 16, 0, 2);
    }
  };
  floatx4_t acc[TMAX];
#pragma unroll
  for (int t = 0; t < TMAX; ++t) acc[t] = floatx4_t{0.f, 0.f, 0.f, 0.f};
  issue(0);
  if (U > 1) issue(1);
#pragma unroll
  for (int t = 0; t < TMAX; ++t) {
    if (t >= T) break;  // uniform
#pragma unroll
    for (int s = 0; s < NSPAN; ++s) {
      const int u = t * NSPAN + s;
      // this wave's loads of unit u have landed (unit u + 1 still in flight), then every wave's
      if (u + 1 < U) wait_vm<kUnitLoads>();
      else wait_vm<0>();
      ring_barrier();
      const unsigned char* buf = lds_u + (u & 1) * kUnitBytes;
      bf16x8_t bw[kUnitSteps];  // B operand: weight row fr of the tile
#pragma unroll
      for (int j = 0; j < kUnitSteps; ++j)
        bw[j] = *reinterpret_cast<const bf16x8_t*>(
            buf + fr * kUnitRowBytes + 2 * (32 * (kUnitSteps * wave + j) + 8 * grp));
#pragma unroll
      for (int j = 0; j < kUnitSteps; ++j)
        acc[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(xa[s][j], bw[j], acc[t], 0, 0, 0);
      if (u + 2 < U) {
        ring_barrier();  // every wave is done reading buffer u & 1
        issue(u + 2);
      }
    }
  }
  // the waves' partials summed in wave order: red[w][t][lane], then res
  __syncthreads();
  floatx4_t* red = reinterpret_cast<floatx4_t*>(lds_u);
  float* res = reinterpret_cast<float*>(lds_u + kUnitWaves * TMAX * kWave * 16);
#pragma unroll
  for (int t = 0; t < TMAX; ++t)
    if (t < T) red[(wave * TMAX + t) * kWave + lane] = acc[t];
  __syncthreads();
  if (tid < T * kWave) {
    const int t = tid >> 6, l = tid & (kWave - 1);
    floatx4_t v = red[t * kWave + l];
#pragma unroll
    for (int w = 1; w < kUnitWaves; ++w) v += red[(w * TMAX + t) * kWave + l];
    // C layout: lane l holds weight row (l & 15) of the tile and x rows 4 (l >> 4) + e
#pragma unroll
    for (int e = 0; e < 4; ++e) res[(16 * t + (l & 15)) * 16 + 4 * (l >> 4) + e] = v[e];
  }
  __syncthreads();
  return res;
}

template <int NSPAN>  // d_model / 2048
__global__ __launch_bounds__(kUnitThreads) void gu_unit_kernel(
    const uint16_t* __restrict__ xp, int B, const uint16_t* __restrict__ wg,
    const uint16_t* __restrict__ wu, int d, int F, int hs, int np, int sp,
    uint16_t* __restrict__ hhi, uint16_t* __restrict__ hlo) {
  extern __shared__ __attribute__((aligned(16))) unsigned char lds_u[];
  const int tid = threadIdx.x, lane = tid & (kWave - 1);
  const int n0 = blockIdx.x * np;
  // x operand: token rows (rows past B are zero in xp)
  bf16x8_t xa[NSPAN][kUnitSteps];
  unit_x<NSPAN>(xa, xp + (size_t)(lane & 15) * d, true);
  const float* res = unit_pass<NSPAN, kUnitTiles>(
      lds_u, (2 * np + 15) >> 4,
      [&](int r) -> const uint16_t* {
        return r < np       ? wg + (size_t)min(n0 + r, F - 1) * d
               : r < 2 * np ? wu + (size_t)min(n0 + r - np, F - 1) * d
                            : nullptr;
      },
      xa);
  // h at the segment's positions [0, sp), as gu_frag_kernel writes it: neuron n0 + j, zero past
  // the segment's rows, past d_ff and for the padding tokens
  for (int i = tid; i < 16 * sp; i += kUnitThreads) {
    const int m = i / sp, j = i - m * sp;
    const bool real = j < np && n0 + j < F && m < B;
    store_h(hhi, hlo, (size_t)m * hs + (size_t)blockIdx.x * sp + j,
            real ? silu(res[j * 16 + m]) * res[(np + j) * 16 + m] : 0.f);
  }
  if (blockIdx.x == gridDim.x - 1) zero_h_tail(hhi, hlo, hs, gridDim.x * sp, 16);
}

// ---- per-token sparse gate/up of at most 4 tokens on the exact input (threshold, top-k gate pass,
// top-k keyed pass, every neuron kept), d_model a multiple of 2048, on the unit pipeline: the
// three bf16 pieces of the four tokens are the 12 rows of one MFMA operand tile (row 4 p + m), so
// the whole input stays in registers. Phase A streams the segment's gate rows, phase B the up rows
// of the tokens' union; keep decisions, lists and h as cats_frag_kernel forms them. A row's sum is
// its three pieces' sums added in piece order. With every neuron kept the gate and up rows go in
// one pass (each row's result is the same wherever it sits in the sequence), so a threshold below
// 0 still gives the dense result bit for bit.
constexpr int kCatsUnitTokens = 4;
constexpr int kCatsUnitTiles = (kSegN + 15) / 16;  // 16-row tiles of one phase (4)
constexpr int kModeThr = 0, kModeAct = 1, kModeKeyed = 2, kModeAll = 3;

__device__ __forceinline__ float piece_sum(const float* res, int row, int m) {
  return (res[row * 16 + m] + res[row * 16 + 4 + m]) + res[row * 16 + 8 + m];
}

template <int NSPAN, int MODE>
__global__ __launch_bounds__(kUnitThreads) void cats_unit_kernel(
    const uint16_t* __restrict__ xp, int B, const uint16_t* __restrict__ wg,
    const uint16_t* __restrict__ wu, int d, int F, int np, float t, float* __restrict__ act,
    const unsigned long long* __restrict__ cut, uint16_t* __restrict__ hhi,
    uint16_t* __restrict__ hlo, int hs, int sp, int32_t* __restrict__ uidx,
    int32_t* __restrict__ ucnt, int32_t* __restrict__ bidx, int32_t* __restrict__ bcnt) {
  extern __shared__ __attribute__((aligned(16))) unsigned char lds_u[];
  __shared__ float s_a[kCatsUnitTokens][kSegPad];         // a = SiLU(g) per token and position
  __shared__ unsigned long long s_keep[kCatsUnitTokens];  // kept positions per token
  __shared__ int s_u[kSegPad];                            // union positions, ascending
  __shared__ int s_nu;
  const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid >> 6;
  const int seg = blockIdx.x, nseg = gridDim.x;
  const int r0 = seg * np;
  const int nr = min(np, F - r0);  // neurons of this segment (>= 1)
  constexpr int kMpad = 16;        // rows of xp per piece and of h

  // x operand: row 4 p + m = piece p of token m (rows 12..15 and tokens past B: zero)
  bf16x8_t xa[NSPAN][kUnitSteps];
  {
    const int fr = lane & 15, pc = fr >> 2, m = fr & 3;
    const bool ok = fr < 12 && m < B;
    unit_x<NSPAN>(xa, xp + ((size_t)(ok ? pc : 0) * kMpad + (ok ? m : 0)) * d, ok);
  }

  if (MODE == kModeAll) {  // gate rows [0, np), up rows [np, 2 np) in one pass
    const float* res = unit_pass<NSPAN, kUnitTiles>(
        lds_u, (2 * np + 15) >> 4,
        [&](int r) -> const uint16_t* {
          return r < np       ? wg + (size_t)(r0 + min(r, nr - 1)) * d
                 : r < 2 * np ? wu + (size_t)(r0 + min(r - np, nr - 1)) * d
                              : nullptr;
        },
        xa);
    for (int i = tid; i < kMpad * sp; i += kUnitThreads) {
      const int m = i / sp, k = i - m * sp;
      const float h = (m < B && k < nr) ? silu(piece_sum(res, k, m)) * piece_sum(res, np + k, m) : 0.f;
      store_h(hhi, hlo, (size_t)m * hs + (size_t)seg * sp + k, h);
    }
    // the kept list of every neuron, as the threshold path writes it for t < 0
    if (tid < nr) uidx[seg * sp + tid] = r0 + tid;
    if (tid == 0) ucnt[seg] = nr;
    if (seg == nseg - 1) zero_h_tail(hhi, hlo, hs, nseg * sp, kMpad);
    return;
  }

  // ---- phase A: the gate (threshold mode and the top-k gate pass) or the stored activations
  if (MODE != kModeKeyed) {
    const float* res = unit_pass<NSPAN, kCatsUnitTiles>(
        lds_u, (np + 15) >> 4,
        [&](int r) -> const uint16_t* {
          return r < np ? wg + (size_t)(r0 + min(r, nr - 1)) * d : nullptr;
        },
        xa);
    for (int i = tid; i < kCatsUnitTokens * kSegPad; i += kUnitThreads) {
      const int m = i / kSegPad, j = i - m * kSegPad;
      if (j < np) {
        const float a = silu(piece_sum(res, j, m));
        if (MODE == kModeAct) {
          if (m < B && j < nr) act[(size_t)m * F + r0 + j] = a;
        } else {
          s_a[m][j] = a;
        }
      }
    }
    if (MODE == kModeAct) return;  // uniform
  } else {
    for (int i = tid; i < kCatsUnitTokens * kSegPad; i += kUnitThreads) {
      const int m = i / kSegPad, j = i - m * kSegPad;
      s_a[m][j] = (m < B && j < nr) ? act[(size_t)m * F + r0 + j] : 0.f;
    }
  }
  __syncthreads();

  // ---- keep decisions per token (a wave ballot over the segment's positions), per-token lists
  if (wave < kCatsUnitTokens) {
    const int m = wave;
    const float a = s_a[m][lane];
    bool keep = false;
    if (m < B && lane < nr) {
      if (MODE == kModeKeyed) keep = topk_key(a, r0 + lane) >= cut[m];
      else keep = fabsf(a) > t;
    }
    const unsigned long long mk = __ballot(keep);
    if (lane == 0) s_keep[m] = mk;
    if (m < B && bidx != nullptr) {
      if (keep) bidx[((size_t)m * nseg + seg) * sp + __popcll(mk & ((1ull << lane) - 1ull))] = r0 + lane;
      if (lane == 0) bcnt[m * nseg + seg] = __popcll(mk);
    }
  }
  __syncthreads();
  // ---- union of the tokens' kept positions, ascending
  if (wave == 0) {
    unsigned long long un = 0ull;
    for (int m = 0; m < B && m < kCatsUnitTokens; ++m) un |= s_keep[m];
    const bool in = (un >> lane) & 1ull;
    const int pos = __popcll(un & ((1ull << lane) - 1ull));
    if (in) {
      s_u[pos] = lane;
      uidx[seg * sp + pos] = r0 + lane;
    }
    if (lane == 0) {
      s_nu = __popcll(un);
      ucnt[seg] = __popcll(un);
    }
  }
  __syncthreads();
  const int nu = s_nu;

  // ---- phase B: the up rows of the union only; h = a u where the token keeps the neuron
  const float* res = nullptr;
  if (nu > 0)  // uniform
    res = unit_pass<NSPAN, kCatsUnitTiles>(
        lds_u, (nu + 15) >> 4,
        [&](int k) -> const uint16_t* { return k < nu ? wu + (size_t)(r0 + s_u[k]) * d : nullptr; },
        xa);
  for (int i = tid; i < kMpad * sp; i += kUnitThreads) {
    const int m = i / sp, k = i - m * sp;
    float h = 0.f;
    if (m < B && k < nu) {
      const int j = s_u[k];
      if ((s_keep[m] >> j) & 1ull) h = s_a[m][j] * piece_sum(res, k, m);
    }
    store_h(hhi, hlo, (size_t)m * hs + (size_t)seg * sp + k, h);  // 0 past nu
  }
  if (seg == nseg - 1) zero_h_tail(hhi, hlo, hs, nseg * sp, kMpad);
}

// ---- the operand-order pipeline of the other batches (any d_model % 256 == 0, up to 64 tokens): one
// workgroup of eight waves per segment. The weight rows come through registers, two blocks of 256
// columns ahead, into two LDS buffers (whole runs of a row per request; the 16 rows of an MFMA
// operand from LDS); wave w multiplies columns 32 w .. + 31 of every block by the x pieces, which
// it reads from L2 in operand order into registers. The eight waves' sums (an eighth of K each) are
// added in wave order. A row's result does not depend on its place in the sequence. Bound by HBM; the
// earlier kernels copied the pieces (up to 4 x 3 token tiles) through an LDS ring next to the weights
// in every workgroup, which cost more LDS writes than the weights themselves from 17 tokens on.
// Gate/up, ring -> here: threshold call 14336 x 4096 at 40 tokens 91 -> 68 us, 22671 x 8192 at 40
// tokens 342 -> 209; dense 15104 x 4608 at 16 tokens 66 -> 43; even at 14336 x 4096 and 16 tokens or
// fewer in the dense modes (39 -> 39), where the weights alone fill the time; threshold mode 48.5 -> 45.5
// there. Four blocks ahead instead of two: 47.5, eight: 51; 1024 threads on 512 columns: 48.5.
constexpr int kFrThreads = 512;
constexpr int kFrWaves = kFrThreads / kWave;
constexpr int kFrK = 256;                       // columns per block: one K step per wave
constexpr int kFrCpr = kFrK / 8;                // 16-byte chunks per row and block
constexpr int kFrPitch = kFrK * 2 + 16;         // the 16 rows of an operand read: all banks
constexpr int kFrRowStep = kFrThreads / kFrCpr; // rows between a thread's loads (16)
static_assert(kFrK / 32 == kFrWaves && kFrRowStep == 16, "one K step per wave, one row tile per load");

template <int MT, int RT>
struct FrLds {
  static constexpr int kBuf = 16 * RT * kFrPitch;
  static constexpr int kRed = kFrWaves * RT * kWave * 16;            // one token tile's partials
  // token pitch of the results: the 64 rows that a wave then reads at one token in 16 banks of 64
  static constexpr int kResPitch = 16 * MT + 4;
  static constexpr int kRes = 16 * RT * kResPitch * 4;
  static constexpr int kBytes = 2 * kBuf > kRed + kRes ? 2 * kBuf : kRed + kRes;
};

// nrows (<= 16 RT) rows from row_of(r), r < nrows; returns res[kResPitch * row + token] in lds. xf: px
// pieces in operand order (prep_frag_kernel).
template <int PX, int MT, int RT, class RowOf>
__device__ __forceinline__ const float* frag_pass(unsigned char* lds, int nrows, RowOf row_of,
                                                  const uint4* __restrict__ xf, int d) {
  using S = FrLds<MT, RT>;
  const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid >> 6;
  const int fr = lane & 15, grp = lane >> 4;
  const int T = (nrows + 15) >> 4;               // row tiles
  const int nblk = d / kFrK;                     // d % 256 == 0
  const int ch = tid % kFrCpr, row0 = tid / kFrCpr;
  const uint4* src[RT];
#pragma unroll
  for (int i = 0; i < RT; ++i)  // rows past the last of a tile: the last one again, never used
    src[i] = reinterpret_cast<const uint4*>(row_of(min(16 * i + row0, nrows - 1))) + ch;
  constexpr int D = 2;  // blocks in flight, as many as LDS and x buffers
  uint4 wr[D][RT];
  auto load_w = [&](uint4(&r)[RT], int b) {
#pragma unroll
    for (int i = 0; i < RT; ++i)
      if (i < T) r[i] = ld_stream(src[i] + b * kFrCpr);
  };
  uint4 xa[2][PX][MT];
  auto load_x = [&](uint4(&r)[PX][MT], int b) {
#pragma unroll
    for (int p = 0; p < PX; ++p)
#pragma unroll
      for (int mt = 0; mt < MT; ++mt)
        r[p][mt] = xf[(((size_t)(b * kFrWaves + wave) * PX + p) * MT + mt) * kWave + lane];
  };
  floatx4_t acc[RT][MT];
#pragma unroll
  for (int t = 0; t < RT; ++t)
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) acc[t][mt] = floatx4_t{0.f, 0.f, 0.f, 0.f};
  auto step = [&](uint4(&wcur)[RT], uint4(&xcur)[PX][MT], uint4(&xnext)[PX][MT],
                  int b) {
    unsigned char* buf = lds + (b & 1) * S::kBuf;
#pragma unroll
    for (int i = 0; i < RT; ++i)
      if (i < T) *reinterpret_cast<uint4*>(buf + (16 * i + row0) * kFrPitch + 16 * ch) = wcur[i];
    if (b + D < nblk) load_w(wcur, b + D);
    if (b + 1 < nblk) load_x(xnext, b + 1);
    ring_barrier();  // block b is in its buffer; every wave is done reading block b - 1
    // every tile of the class, also those past T (stale rows, never used): branches around a tile's
    // products would split the block between the MFMAs and what reads their results
    bf16x8_t bw[RT];
#pragma unroll
    for (int t = 0; t < RT; ++t)
      bw[t] = *reinterpret_cast<const bf16x8_t*>(buf + (16 * t + fr) * kFrPitch + 64 * wave + 16 * grp);
#pragma unroll
    for (int p = PX - 1; p >= 0; --p)
#pragma unroll
      for (int t = 0; t < RT; ++t)
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
          acc[t][mt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(xcur[p][mt]), bw[t], acc[t][mt], 0, 0, 0);
  };
#pragma unroll
  for (int u = 0; u < D; ++u)
    if (u < nblk) load_w(wr[u], u);
  load_x(xa[0], 0);
  for (int b = 0; b < nblk; b += D) {
#pragma unroll
    for (int u = 0; u < D; ++u)
      if (b + u < nblk) step(wr[u], xa[u], xa[1 - u], b + u);
  }
  // the waves' totals, one token tile at a time
  floatx4_t* red = reinterpret_cast<floatx4_t*>(lds);
  float* res = reinterpret_cast<float*>(lds + S::kRed);
#pragma unroll
  for (int mt = 0; mt < MT; ++mt) {
    __syncthreads();
#pragma unroll
    for (int t = 0; t < RT; ++t)
      if (t < T) red[(wave * RT + t) * kWave + lane] = acc[t][mt];
    __syncthreads();
    for (int i = tid; i < T * kWave; i += kFrThreads) {
      floatx4_t v = red[i];
#pragma unroll
      for (int w = 1; w < kFrWaves; ++w) v += red[w * RT * kWave + i];
      // C layout: lane l holds weight row l & 15 of the tile and tokens 4 (l >> 4) + e
      const int t = i >> 6, l = i & (kWave - 1);
      *reinterpret_cast<floatx4_t*>(&res[(16 * t + (l & 15)) * S::kResPitch + 16 * mt + 4 * (l >> 4)]) = v;
    }
  }
  __syncthreads();
  return res;
}

// Dense gate/up on the bf16-rounded input: gate rows [0, np), up rows [np, 2 np) in one pass.
template <int MT, int RT>
__global__ __launch_bounds__(kFrThreads, 2) void gu_frag_kernel(
    const uint4* __restrict__ xf, int B, const uint16_t* __restrict__ wg,
    const uint16_t* __restrict__ wu, int d, int F, int hs, int np, int sp,
    uint16_t* __restrict__ hhi, uint16_t* __restrict__ hlo) {
  extern __shared__ __attribute__((aligned(16))) unsigned char lds_u[];
  constexpr int kPitch = FrLds<MT, RT>::kResPitch;
  const int n0 = blockIdx.x * np;
  const float* res = frag_pass<1, MT, RT>(
      lds_u, 2 * np,
      [&](int r) {
        return r < np ? wg + (size_t)min(n0 + r, F - 1) * d : wu + (size_t)min(n0 + r - np, F - 1) * d;
      },
      xf, d);
  for (int i = threadIdx.x; i < 16 * MT * sp; i += kFrThreads) {
    const int m = i / sp, j = i - m * sp;
    const bool real = j < np && n0 + j < F && m < B;
    store_h(hhi, hlo, (size_t)m * hs + (size_t)blockIdx.x * sp + j,
            real ? silu(res[j * kPitch + m]) * res[(np + j) * kPitch + m] : 0.f);
  }
  if (blockIdx.x == gridDim.x - 1) zero_h_tail(hhi, hlo, hs, gridDim.x * sp, 16 * MT);
}

// Per-token sparse gate/up on the exact input, and every neuron kept (kModeAll: the dense and condensed
// FFN of small batches, gate and up rows in one pass; a row's result is the same wherever it sits,
// so a threshold below 0 gives the dense result bit for bit). The modes are those of
// cats_unit_kernel above.
// RT: row tiles of a segment's np rows, or of its 2 np (kModeAll).
template <int MT, int RT, int MODE>
__global__ __launch_bounds__(kFrThreads, 2) void cats_frag_kernel(
    const uint4* __restrict__ xf, int B, const uint16_t* __restrict__ wg,
    const uint16_t* __restrict__ wu, int d, int F, int np, float t, float* __restrict__ act,
    const unsigned long long* __restrict__ cut, uint16_t* __restrict__ hhi,
    uint16_t* __restrict__ hlo, int hs, int sp, int32_t* __restrict__ uidx,
    int32_t* __restrict__ ucnt, int32_t* __restrict__ bidx, int32_t* __restrict__ bcnt) {
  constexpr int kMpad = 16 * MT, kPitch = FrLds<MT, RT>::kResPitch;
  extern __shared__ __attribute__((aligned(16))) unsigned char lds_u[];
  __shared__ float s_a[kMpad][kSegPad];         // a = SiLU(g) per token and position
  __shared__ unsigned long long s_keep[kMpad];  // kept positions per token
  __shared__ int s_u[kSegPad];                  // union positions, ascending
  const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid >> 6;
  const int seg = blockIdx.x, nseg = gridDim.x;
  const int r0 = seg * np;
  const int nr = min(np, F - r0);  // neurons of this segment (>= 1)

  if (MODE == kModeAll) {
    const float* res = frag_pass<3, MT, RT>(
        lds_u, 2 * np,
        [&](int r) {
          return r < np ? wg + (size_t)(r0 + min(r, nr - 1)) * d : wu + (size_t)(r0 + min(r - np, nr - 1)) * d;
        },
        xf, d);
    for (int i = tid; i < kMpad * sp; i += kFrThreads) {
      const int m = i / sp, k = i - m * sp;
      const float h = (m < B && k < nr) ? silu(res[k * kPitch + m]) * res[(np + k) * kPitch + m] : 0.f;
      store_h(hhi, hlo, (size_t)m * hs + (size_t)seg * sp + k, h);
    }
    // the kept list of every neuron, as the threshold path writes it for t < 0
    if (tid < nr) uidx[seg * sp + tid] = r0 + tid;
    if (tid == 0) ucnt[seg] = nr;
    if (seg == nseg - 1) zero_h_tail(hhi, hlo, hs, nseg * sp, kMpad);
    return;
  }

  // ---- phase A: the gate (threshold mode and the top-k gate pass) or the stored activations
  if (MODE != kModeKeyed) {
    const float* res = frag_pass<3, MT, RT>(
        lds_u, np, [&](int r) { return wg + (size_t)(r0 + min(r, nr - 1)) * d; }, xf, d);
    for (int i = tid; i < kMpad * np; i += kFrThreads) {
      const int j = i % np, m = i / np;
      const float a = silu(res[j * kPitch + m]);
      if (MODE == kModeAct) {
        if (m < B && j < nr) act[(size_t)m * F + r0 + j] = a;
      } else {
        s_a[m][j] = a;
      }
    }
    if (MODE == kModeAct) return;  // uniform
  } else {
    for (int i = tid; i < kMpad * kSegPad; i += kFrThreads) {
      const int m = i / kSegPad, j = i % kSegPad;
      s_a[m][j] = (m < B && j < nr) ? act[(size_t)m * F + r0 + j] : 0.f;
    }
  }
  __syncthreads();

  // ---- keep decisions per token (a wave ballot over the segment's positions), per-token lists
  for (int m = wave; m < kMpad; m += kFrWaves) {
    bool keep = false;
    if (m < B && lane < nr) {
      const float a = s_a[m][lane];
      if (MODE == kModeKeyed) keep = topk_key(a, r0 + lane) >= cut[m];
      else keep = fabsf(a) > t;
    }
    const unsigned long long mk = __ballot(keep);
    if (lane == 0) s_keep[m] = mk;
    if (m < B && bidx != nullptr) {
      if (keep) bidx[((size_t)m * nseg + seg) * sp + __popcll(mk & ((1ull << lane) - 1ull))] = r0 + lane;
      if (lane == 0) bcnt[m * nseg + seg] = __popcll(mk);
    }
  }
  __syncthreads();
  // ---- union of the tokens' kept positions, ascending: every wave forms it for itself
  unsigned long long un = lane < B ? s_keep[lane] : 0ull;
  static_assert(kMpad <= kWave, "a lane per token");
  for (int off = kWave / 2; off > 0; off >>= 1) un |= __shfl_xor(un, off, kWave);
  const int nu = __popcll(un);
  const int pos = __popcll(un & ((1ull << lane) - 1ull));
  if ((un >> lane) & 1ull) {
    s_u[pos] = lane;  // the same value from every wave
    if (wave == 0) uidx[seg * sp + pos] = r0 + lane;
  }
  if (tid == 0) ucnt[seg] = nu;
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");  // the wave's own list, read across its lanes

  // ---- phase B: the up rows of the union only; h = a u where the token keeps the neuron
  const float* res = nullptr;
  if (nu > 0)  // uniform
    res = frag_pass<3, MT, RT>(
        lds_u, nu, [&](int k) { return wu + (size_t)(r0 + s_u[k]) * d; }, xf, d);
  for (int i = tid; i < kMpad * sp; i += kFrThreads) {
    const int m = i / sp, k = i - m * sp;
    float h = 0.f;
    if (m < B && k < nu) {
      const int j = s_u[k];
      if ((s_keep[m] >> j) & 1ull) h = s_a[m][j] * res[k * kPitch + m];
    }
    store_h(hhi, hlo, (size_t)m * hs + (size_t)seg * sp + k, h);  // 0 past nu
  }
  if (seg == nseg - 1) zero_h_tail(hhi, hlo, hs, nseg * sp, kMpad);
}

// ---- down product: Y_partial[rho][m][c] over one 256-column tile and one range of 64-row blocks.
// Block b is positions 64 b .. + 63 of the segment layout (segment s owns positions s sp .. +
// sp - 1, sp in {16, 32, 48, 64}). Whole segments (GATHER = 0, the dense gate/up kernel): position
// s sp + k is W_down row s np + k for k < np (and below d_ff). Kept lists (GATHER = 1): it is row
// uidx[s sp + k] for k < ucnt[s]. Any other position has no row (h = 0 there; W_down row 0 is
// loaded, an L2 hit). The 64-row blocks of whole segments measured faster than blocks of 64
// consecutive neurons (dense 16-token pass at the Llama-3-8B layer: 22.6 against 27.2 us).
// Slot: the block's 64 W_down rows over the tile (512 bytes each; chunk c of row r at
// c ^ 2 ((r / 8) % 4), so the 16-bit B-operand gathers of one instruction touch 32 banks), then
// the hi/lo h fragments in A-operand lane order. Wave w: columns 32 w .. + 31 (two 16-column tiles).
template <int MT>
struct DnShape {
  static constexpr int kWBytes = kDnBlock * kDnCols * 2;             // 32 KiB
  static constexpr int kHBytes = 2 * MT * 2 * kWave * 16;            // hi/lo x tiles x 2 K steps
  static constexpr int kSlotBytes = kWBytes + kHBytes;
  static constexpr int kPieces = kSlotBytes / 16;
  static constexpr int kWPieces = kWBytes / 16;
  static constexpr int kLoads = (kPieces + kBT - 1) / kBT;
  static constexpr int kFullWaves = (kPieces - (kLoads - 1) * kBT) / kWave;
  static constexpr int kSlotsMax = kLdsRing / kSlotBytes;
  static constexpr int kSlots = kSlotsMax > 4 ? 4 : kSlotsMax;
  static_assert(kPieces % kWave == 0 && kWPieces % kWave == 0, "whole wave instructions");
  static_assert(kSlots >= 3 && kSlots <= 4, "two or three blocks in flight, wait_later's counts");
};

__device__ __forceinline__ int dr_pos(int row, int chunk) { return chunk ^ (((row >> 3) & 3) << 1); }

template <int MT, int GATHER>
__global__ __launch_bounds__(kBT) void down_ring_kernel(
    const uint16_t* __restrict__ hhi, const uint16_t* __restrict__ hlo, int hs,
    const uint16_t* __restrict__ wd, int d, int F, int B, int nblocks, int gr, int nseg, int np,
    int sp, const int32_t* __restrict__ uidx, const int32_t* __restrict__ ucnt,
    float* __restrict__ part) {
  using DS = DnShape<MT>;
  __shared__ __attribute__((aligned(16))) unsigned char ring[DS::kSlots * DS::kSlotBytes];
  __shared__ int s_rows[16 * kDnBlock];  // the range's W_down row indices (gathered blocks)
  const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid >> 6;
  // workgroups go to the eight XCDs in turn (id % 8); when the grid divides evenly, XCD j takes
  // the consecutive (tile, range) indices [j N / 8, (j + 1) N / 8), so the column tiles of a
  // range share one L2 and its h fragments come from HBM once
  const int ncols = d / kDnCols, N = ncols * gr;
  const int L = blockIdx.x;
  const int idx = (N % 8 == 0) ? (L % 8) * (N / 8) + L / 8 : L;
  const int c0 = (idx % ncols) * kDnCols, rho = idx / ncols;
  const int b_lo = (int)(((long long)nblocks * rho) / gr);
  const int nb = (int)(((long long)nblocks * (rho + 1)) / gr) - b_lo;

  {  // row indices of the range's blocks (at most 16 blocks of 64 positions)
    for (int i = tid; i < nb * kDnBlock; i += kBT) {
      const int pos = b_lo * kDnBlock + i, s = pos / sp, k = pos % sp;
      // a position past its segment's rows (h = 0 there) reads W_down row 0, an L2 hit; the
      // kept lists give the rows of a gathered segment, neuron s np + k those of a whole one
      int n = 0;
      if (GATHER) n = (s < nseg && k < ucnt[s]) ? uidx[s * sp + k] : 0;
      else if (s < nseg && k < np && s * np + k < F) n = s * np + k;
      s_rows[i] = n;
    }
    __syncthreads();
  }
  // this thread's pieces of a block: piece g = q * 512 + tid; below kWPieces: W_down row g / 32,
  // position g % 32 holding chunk dr_pos(row, position) of the tile's columns; above: h fragment
  // (which, mt, step, lane) = hg / (MT 128), (hg / 128) % MT, (hg / 64) % 2, hg % 64
  const bool full = wave < DS::kFullWaves;
  int lds_off[DS::kLoads], wrow[DS::kLoads], wchunk[DS::kLoads];
  const uint16_t* hsrc[DS::kLoads];
#pragma unroll
  for (int q = 0; q < DS::kLoads; ++q) {
    const int g = min(q * kBT + tid, DS::kPieces - 1);
    lds_off[q] = (q * kBT + wave * kWave) * 16;
    if (g < DS::kWPieces) {
      wrow[q] = g >> 5;
      wchunk[q] = dr_pos(g >> 5, g & 31);
      hsrc[q] = nullptr;
    } else {
      const int hg = g - DS::kWPieces;
      const int which = hg / (MT * 128), mt = (hg / 128) % MT, st = (hg >> 6) & 1, l = hg & 63;
      wrow[q] = -1;
      wchunk[q] = 0;
      hsrc[q] = (which ? hlo : hhi) + (size_t)(16 * mt + (l & 15)) * hs + 32 * st + 8 * (l >> 4);
    }
  }
  auto issue = [&](unsigned char* slot, int b) {
    const int blk = b_lo + b;
#pragma unroll
    for (int q = 0; q < DS::kLoads; ++q) {
      if (q == DS::kLoads - 1 && !full) break;  // wave-uniform
      auto* lp = reinterpret_cast<__attribute__((address_space(3))) void*>(
          reinterpret_cast<size_t>(slot + lds_off[q]));
      const int g0 = __builtin_amdgcn_readfirstlane(q * kBT + wave * kWave);
      if (g0 < DS::kWPieces) {
        const int n = s_rows[b * kDnBlock + wrow[q]];
        __builtin_amdgcn_global_load_lds(static_cast<const void*>(wd + (size_t)n * d + c0 + 8 * wchunk[q]), lp, 16, 0, 2);
      } else {
        __builtin_amdgcn_global_load_lds(static_cast<const void*>(hsrc[q] + (size_t)blk * kDnBlock), lp, 16, 0, 0);
      }
    }
  };

  const int nbv = lane & 15, gq = lane >> 4;
  floatx4_t acc[2][MT];
#pragma unroll
  for (int j = 0; j < 2; ++j)
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) acc[j][mt] = floatx4_t{0.f, 0.f, 0.f, 0.f};
  auto compute = [&](const unsigned char* slot) {
#pragma unroll
    for (int st = 0; st < 2; ++st) {
      bf16x8_t ahi[MT], alo[MT];
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) {
        ahi[mt] = as_bf16x8(*reinterpret_cast<const uint4*>(slot + DS::kWBytes + 16 * (((0 * MT + mt) * 2 + st) * kWave + lane)));
        alo[mt] = as_bf16x8(*reinterpret_cast<const uint4*>(slot + DS::kWBytes + 16 * (((1 * MT + mt) * 2 + st) * kWave + lane)));
      }
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        const int col = 32 * wave + 16 * j + nbv;
        uint32_t bw[4];
#pragma unroll
        for (int jj = 0; jj < 4; ++jj) {
          const int ra = 32 * st + 8 * gq + 2 * jj, rb = ra + 1;
          const uint32_t e0 = *reinterpret_cast<const uint16_t*>(slot + ra * 512 + 16 * dr_pos(ra, col >> 3) + 2 * (col & 7));
          const uint32_t e1 = *reinterpret_cast<const uint16_t*>(slot + rb * 512 + 16 * dr_pos(rb, col >> 3) + 2 * (col & 7));
          bw[jj] = e0 | (e1 << 16);
        }
        const bf16x8_t bop = as_bf16x8(make_uint4(bw[0], bw[1], bw[2], bw[3]));
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) {
          acc[j][mt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ahi[mt], bop, acc[j][mt], 0, 0, 0);
          acc[j][mt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(alo[mt], bop, acc[j][mt], 0, 0, 0);
        }
      }
    }
  };
#pragma unroll
  for (int p = 0; p < DS::kSlots - 1; ++p)
    if (p < nb) issue(ring + p * DS::kSlotBytes, p);
  int slot = 0, refill = DS::kSlots - 1;
  for (int b = 0; b < nb; ++b) {
    const int later = min(DS::kSlots - 2, nb - 1 - b);
    if (full) wait_later<DS::kLoads>(later);
    else wait_later<DS::kLoads - 1>(later);
    ring_barrier();
    if (b + DS::kSlots - 1 < nb) issue(ring + refill * DS::kSlotBytes, b + DS::kSlots - 1);
    compute(ring + slot * DS::kSlotBytes);
    slot = slot + 1 == DS::kSlots ? 0 : slot + 1;
    refill = refill + 1 == DS::kSlots ? 0 : refill + 1;
  }

  // C layout: lane holds column c0 + 32 wave + 16 j + lane % 16 and tokens 4 (lane / 16) + r
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    const int c = c0 + 32 * wave + 16 * j + nbv;
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int m = 16 * mt + 4 * gq + r;
        if (m < B) part[((size_t)rho * B + m) * d + c] = acc[j][mt][r];
      }
  }
}

int batch_mt(int B) { return (B + 15) / 16; }

constexpr int kSegSmall = 32;  // segments of at most this many neurons take fewer row tiles
// the dense unit kernel takes one 16-token tile and d_model = 2048, 4096, 6144 or 8192
bool gu_unit_ok(int B, int d) { return B <= 16 && d % kUnitK == 0 && d <= 4 * kUnitK; }

// Neurons per segment at most. gu_frag_kernel<1 or 2, RT> fits twice on a CU with short segments, so
// that one workgroup's loads run through the other's prologue and epilogue, which a short row does not
// outweigh: at 24 tokens 1024 x 38000 59.7 us against 67.6 with full segments, 1536 x 14336 41.9 against
// 43.2, 2048 x 28672 76.4 against 84.3 (x 14336 46.5 against 46.1). Not where full segments hold 48
// neurons or fewer and short ones would waste positions (1024 x 9000 24.2 against 23.6), nor at 40
// tokens, one workgroup per CU either way (1024 x 14336 40.6 against 38.1).
int dense_seg_cap(int px, int B, int d, int F) {
  const bool narrow = (d <= 1536 && F > kSegTarget * 48) || (d <= 2304 && F > kSegTarget * kSegN);
  return px == 1 && B <= 32 && narrow && !gu_unit_ok(B, d) ? kSegSmall : kSegN;
}

}  // namespace

hipError_t launch_prep_pieces3(const float* x, int B, int d, int mpad, uint16_t* xp, hipStream_t stream) {
  klaunch(prep_pieces_kernel<3>, mpad, 256, 0, stream, x, B, d, mpad, -1.f, xp);
  return hipGetLastError();
}

bool batch_path_ok(int B, int d, int F) {
  return B >= 2 && B <= 64 && d % kDnCols == 0 && d <= 8192 && F >= 1 && F <= 65536;
}

BatchLayout batch_layout(int B, int d, int F, int px) {
  BatchLayout L{};
  const int mt = batch_mt(B);
  L.mpad = 16 * mt;
  L.px = px;
  const int ncols = d / kDnCols;
  // one layout for every mode: segments of np consecutive neurons, each owning sp positions
  // (whole MFMA tiles) of h, the kept list and the down blocks
  const Seg s = seg_of(F, dense_seg_cap(px, B, d, F));
  L.nseg = s.nseg;
  L.np = s.np;
  L.sp = seg_positions(L.np);
  L.nblocks = (L.nseg * L.sp + kDnBlock - 1) / kDnBlock;
  L.hs = L.nblocks * kDnBlock;
  // down ranges: about 256 workgroups in all, at most 16 blocks per range (the gathered row list)
  L.gr = std::max(1, std::min(L.nblocks, 256 / ncols));
  while ((L.nblocks + L.gr - 1) / L.gr > 16) ++L.gr;
  Carve c;
  L.xp = c.take((size_t)px * L.mpad * d * 2);
  L.hhi = c.take((size_t)L.mpad * L.hs * 2);
  L.hlo = c.take((size_t)L.mpad * L.hs * 2);
  L.uidx = c.take((size_t)L.hs * 4);
  L.ucnt = c.take((size_t)L.nseg * 4);
  L.bidx = c.take((size_t)B * L.nseg * L.sp * 4);
  L.bcnt = c.take((size_t)B * L.nseg * 4);
  L.part = c.take((size_t)L.gr * B * d * 4);
  L.total = c.off;
  return L;
}

namespace {

// Lets a kernel take up to `bytes` of dynamic LDS (once per kernel, on its first launch).
hipError_t allow_dynamic_lds(const void* kernel, int bytes) {
  return hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
}

template <int NSPAN>
hipError_t launch_gu_unit_n(const BatchLayout& L, hipStream_t stream, const uint16_t* xp, int B,
                            const uint16_t* wg, const uint16_t* wu, int d, int F, uint16_t* hhi,
                            uint16_t* hlo) {
  static const hipError_t attr =
      allow_dynamic_lds(reinterpret_cast<const void*>(gu_unit_kernel<NSPAN>), kUnitLds);
  if (attr != hipSuccess) return attr;
  klaunch(gu_unit_kernel<NSPAN>, L.nseg, kUnitThreads, (uint32_t)kUnitLds, stream, xp, B, wg, wu, d,
          F, L.hs, L.np, L.sp, hhi, hlo);
  return hipGetLastError();
}
hipError_t launch_gu_unit(const BatchLayout& L, hipStream_t stream, const uint16_t* xp, int B,
                          const uint16_t* wg, const uint16_t* wu, int d, int F, uint16_t* hhi,
                          uint16_t* hlo) {
  switch (d / kUnitK) {
    case 1: return launch_gu_unit_n<1>(L, stream, xp, B, wg, wu, d, F, hhi, hlo);
    case 2: return launch_gu_unit_n<2>(L, stream, xp, B, wg, wu, d, F, hhi, hlo);
    case 3: return launch_gu_unit_n<3>(L, stream, xp, B, wg, wu, d, F, hhi, hlo);
    case 4: return launch_gu_unit_n<4>(L, stream, xp, B, wg, wu, d, F, hhi, hlo);
    default: return hipErrorInvalidValue;
  }
}
template <int MT, int RT>
hipError_t launch_gu_frag_n(const BatchLayout& L, hipStream_t stream, const uint16_t* xp, int B,
                            const uint16_t* wg, const uint16_t* wu, int d, int F, uint16_t* hhi,
                            uint16_t* hlo) {
  constexpr int kLds = FrLds<MT, RT>::kBytes;
  static const hipError_t attr = allow_dynamic_lds(reinterpret_cast<const void*>(gu_frag_kernel<MT, RT>), kLds);
  if (attr != hipSuccess) return attr;
  klaunch((gu_frag_kernel<MT, RT>), L.nseg, kFrThreads, (uint32_t)kLds, stream,
          reinterpret_cast<const uint4*>(xp), B, wg, wu, d, F, L.hs, L.np, L.sp, hhi, hlo);
  return hipGetLastError();
}
template <int MT>
hipError_t launch_gu_frag(const BatchLayout& L, hipStream_t stream, const uint16_t* xp, int B,
                          const uint16_t* wg, const uint16_t* wu, int d, int F, uint16_t* hhi,
                          uint16_t* hlo) {
  return L.np <= kSegSmall ? launch_gu_frag_n<MT, 4>(L, stream, xp, B, wg, wu, d, F, hhi, hlo)
                           : launch_gu_frag_n<MT, kUnitTiles>(L, stream, xp, B, wg, wu, d, F, hhi, hlo);
}

template <int MT, int RT, int MODE>
hipError_t launch_cats_frag_n(const BatchLayout& L, hipStream_t stream, const uint16_t* xp, int B,
                              const uint16_t* wg, const uint16_t* wu, int d, int F, float t, float* act,
                              const unsigned long long* cut, uint16_t* hhi, uint16_t* hlo,
                              int32_t* uidx, int32_t* ucnt, int32_t* bidx, int32_t* bcnt) {
  constexpr int kLds = FrLds<MT, RT>::kBytes;
  static const hipError_t attr =
      allow_dynamic_lds(reinterpret_cast<const void*>(cats_frag_kernel<MT, RT, MODE>), kLds);
  if (attr != hipSuccess) return attr;
  klaunch((cats_frag_kernel<MT, RT, MODE>), L.nseg, kFrThreads, (uint32_t)kLds, stream,
          reinterpret_cast<const uint4*>(xp), B, wg, wu, d, F, L.np, t, act, cut, hhi, hlo, L.hs, L.sp, uidx,
          ucnt, bidx, bcnt);
  return hipGetLastError();
}
template <int MT, int MODE>
hipError_t launch_cats_frag(const BatchLayout& L, hipStream_t stream, const uint16_t* xp, int B,
                            const uint16_t* wg, const uint16_t* wu, int d, int F, float t, float* act,
                            const unsigned long long* cut, uint16_t* hhi, uint16_t* hlo,
                            int32_t* uidx, int32_t* ucnt, int32_t* bidx, int32_t* bcnt) {
  constexpr int kSmall = MODE == kModeAll ? 4 : 2, kLarge = MODE == kModeAll ? kUnitTiles : kCatsUnitTiles;
  return L.np <= kSegSmall
             ? launch_cats_frag_n<MT, kSmall, MODE>(L, stream, xp, B, wg, wu, d, F, t, act, cut, hhi, hlo, uidx,
                                                    ucnt, bidx, bcnt)
             : launch_cats_frag_n<MT, kLarge, MODE>(L, stream, xp, B, wg, wu, d, F, t, act, cut, hhi, hlo, uidx,
                                                    ucnt, bidx, bcnt);
}

// the unit kernel of the exact-input modes: at most 4 tokens, d_model = 2048, 4096, 6144 or 8192
bool cats_unit_ok(int B, int d) {
  return B <= kCatsUnitTokens && d % kUnitK == 0 && d <= 4 * kUnitK;
}
template <int NSPAN, int MODE>
hipError_t launch_cats_unit_n(const BatchLayout& L, hipStream_t stream, const uint16_t* xp, int B,
                              const uint16_t* wg, const uint16_t* wu, int d, int F, float t,
                              float* act, const unsigned long long* cut, uint16_t* hhi,
                              uint16_t* hlo, int32_t* uidx, int32_t* ucnt, int32_t* bidx,
                              int32_t* bcnt) {
  static const hipError_t attr =
      allow_dynamic_lds(reinterpret_cast<const void*>(cats_unit_kernel<NSPAN, MODE>), kUnitLds);
  if (attr != hipSuccess) return attr;
  klaunch(cats_unit_kernel<NSPAN, MODE>, L.nseg, kUnitThreads, (uint32_t)kUnitLds, stream, xp, B, wg,
          wu, d, F, L.np, t, act, cut, hhi, hlo, L.hs, L.sp, uidx, ucnt, bidx, bcnt);
  return hipGetLastError();
}
template <int MODE>
hipError_t launch_cats_unit(const BatchLayout& L, hipStream_t stream, const uint16_t* xp, int B,
                            const uint16_t* wg, const uint16_t* wu, int d, int F, float t,
                            float* act, const unsigned long long* cut, uint16_t* hhi,
                            uint16_t* hlo, int32_t* uidx, int32_t* ucnt, int32_t* bidx,
                            int32_t* bcnt) {
#define SIRIUS_CATS_UNIT(NS)                                                                   \
  case NS:                                                                                     \
    return launch_cats_unit_n<NS, MODE>(L, stream, xp, B, wg, wu, d, F, t, act, cut, hhi, hlo, \
                                        uidx, ucnt, bidx, bcnt);
  switch (d / kUnitK) {
    SIRIUS_CATS_UNIT(1) SIRIUS_CATS_UNIT(2) SIRIUS_CATS_UNIT(3) SIRIUS_CATS_UNIT(4)
    default:
      return hipErrorInvalidValue;
  }
#undef SIRIUS_CATS_UNIT
}

template <int MODE>
hipError_t launch_cats_tb(int B, const BatchLayout& L, hipStream_t stream, const uint16_t* xp,
                          const uint16_t* wg, const uint16_t* wu, int d, int F, float t,
                          float* act, const unsigned long long* cut, uint16_t* hhi, uint16_t* hlo,
                          int32_t* uidx, int32_t* ucnt, int32_t* bidx, int32_t* bcnt) {
  if (cats_unit_ok(B, d))
    return launch_cats_unit<MODE>(L, stream, xp, B, wg, wu, d, F, t, act, cut, hhi, hlo, uidx, ucnt,
                                  bidx, bcnt);
#define SIRIUS_CATS_MT(MTV)                                                                     \
  case MTV:                                                                                     \
    return launch_cats_frag<MTV, MODE>(L, stream, xp, B, wg, wu, d, F, t, act, cut, hhi, hlo,   \
                                       uidx, ucnt, bidx, bcnt);
  if constexpr (MODE == kModeAll) {  // every neuron kept: fewer than 8 tokens
    switch (batch_mt(B)) { SIRIUS_CATS_MT(1) }
  } else {
    switch (batch_mt(B)) { SIRIUS_CATS_MT(1) SIRIUS_CATS_MT(2) SIRIUS_CATS_MT(3) SIRIUS_CATS_MT(4) }
  }
  return hipErrorInvalidValue;
#undef SIRIUS_CATS_MT
}

}  // namespace

hipError_t launch_ffn_batch(const float* x, int B, const uint16_t* wg, const uint16_t* wu,
                            const uint16_t* wd, int d, int F, int mode, float t, float norm_eps,
                            const float* resid, float* y, int32_t* active_idx,
                            int32_t* active_cnt, char* ws, const BatchLayout& L,
                            hipStream_t stream, const float* act,
                            const unsigned long long* cut) {
  if (!batch_path_ok(B, d, F) || L.mpad != 16 * batch_mt(B)) return hipErrorInvalidValue;
  // the segment kernels (gate pass, then the up rows of the kept union) serve every call on the
  // exact input: threshold, top-k, and dense / condensed small batches with every neuron kept
  const bool exact = L.px == 3;
  if (mode != kFfnModeDense && !exact) return hipErrorInvalidValue;
  if (mode == kFfnModeTopK && (act == nullptr || cut == nullptr)) return hipErrorInvalidValue;
  const int mt = L.mpad / 16;
  uint16_t* xp = reinterpret_cast<uint16_t*>(ws + L.xp);
  uint16_t* hhi = reinterpret_cast<uint16_t*>(ws + L.hhi);
  uint16_t* hlo = reinterpret_cast<uint16_t*>(ws + L.hlo);
  int32_t* uidx = reinterpret_cast<int32_t*>(ws + L.uidx);
  int32_t* ucnt = reinterpret_cast<int32_t*>(ws + L.ucnt);
  const bool lists = mode != kFfnModeDense && active_idx != nullptr;
  int32_t* bidx = lists ? reinterpret_cast<int32_t*>(ws + L.bidx) : nullptr;
  int32_t* bcnt = lists ? reinterpret_cast<int32_t*>(ws + L.bcnt) : nullptr;
  float* part = reinterpret_cast<float*>(ws + L.part);
  const bool thr = mode == kFfnModeThreshold, topk = mode == kFfnModeTopK;
  const bool unit = exact ? cats_unit_ok(B, d) : gu_unit_ok(B, d);  // else the operand-order pipeline
  const char* pfx_prep = "batch_prep";
  const char* pfx_gu = topk ? "batch_topk_up"
                       : thr ? "batch_cats_up"
                             : (exact ? "batch_seg_gate_up" : "batch_gate_up");
  const char* pfx_dn = "batch_down";
  const char* pfx_red = "batch_reduce";
  hipError_t e;
  {
    ProfScope prof(pfx_prep, stream);
    if (!unit) e = launch_prep_frag(x, B, d, norm_eps, L.px, reinterpret_cast<char*>(xp), stream);
    else if (L.px == 3) klaunch(prep_pieces_kernel<3>, L.mpad, 256, 0, stream, x, B, d, L.mpad, norm_eps, xp);
    else klaunch(prep_pieces_kernel<1>, L.mpad, 256, 0, stream, x, B, d, L.mpad, norm_eps, xp);
    if (!unit && e != hipSuccess) return e;
    if ((e = hipGetLastError()) != hipSuccess) return e;
  }
  {
    ProfScope prof(pfx_gu, stream);
    if (!exact) {
      if (unit) {
        e = launch_gu_unit(L, stream, xp, B, wg, wu, d, F, hhi, hlo);
      } else {
        switch (mt) {
          case 1: e = launch_gu_frag<1>(L, stream, xp, B, wg, wu, d, F, hhi, hlo); break;
          case 2: e = launch_gu_frag<2>(L, stream, xp, B, wg, wu, d, F, hhi, hlo); break;
          case 3: e = launch_gu_frag<3>(L, stream, xp, B, wg, wu, d, F, hhi, hlo); break;
          default: e = launch_gu_frag<4>(L, stream, xp, B, wg, wu, d, F, hhi, hlo); break;
        }
      }
    } else if (thr) {
      e = launch_cats_tb<kModeThr>(B, L, stream, xp, wg, wu, d, F, t, nullptr, nullptr, hhi, hlo,
                                   uidx, ucnt, bidx, bcnt);
    } else if (topk) {
      e = launch_cats_tb<kModeKeyed>(B, L, stream, xp, wg, wu, d, F, 0.f, const_cast<float*>(act),
                                     cut, hhi, hlo, uidx, ucnt, bidx, bcnt);
    } else {
      e = launch_cats_tb<kModeAll>(B, L, stream, xp, wg, wu, d, F, 0.f, nullptr, nullptr, hhi, hlo,
                                   uidx, ucnt, bidx, bcnt);
    }
    if (e != hipSuccess) return e;
  }
  {
    ProfScope prof(pfx_dn, stream);
    const int grid = (d / kDnCols) * L.gr;
#define SIRIUS_DN(MTV)                                                                                  \
  if (mt == MTV) {                                                                                      \
    if (exact)                                                                                          \
      klaunch(down_ring_kernel<MTV, 1>, grid, kBT, 0, stream, hhi, hlo, L.hs, wd, d, F, B, L.nblocks,   \
              L.gr, L.nseg, L.np, L.sp, uidx, ucnt, part);                                              \
    else                                                                                                \
      klaunch(down_ring_kernel<MTV, 0>, grid, kBT, 0, stream, hhi, hlo, L.hs, wd, d, F, B, L.nblocks,   \
              L.gr, L.nseg, L.np, L.sp, uidx, ucnt, part);                                              \
  }
    SIRIUS_DN(1) SIRIUS_DN(2) SIRIUS_DN(3) SIRIUS_DN(4)
#undef SIRIUS_DN
    if ((e = hipGetLastError()) != hipSuccess) return e;
  }
  ProfScope prof(pfx_red, stream);
  if (lists)
    return launch_reduce(part, L.gr, B, d, resid, y, stream, F, L.nseg, L.sp, bidx, bcnt,
                         active_idx, active_cnt);
  return launch_reduce(part, L.gr, B, d, resid, y, stream);
}

hipError_t launch_batch_act(const float* x, int B, const uint16_t* wg, int d, int F,
                            float norm_eps, float* act, char* ws, const BatchLayout& L,
                            hipStream_t stream) {
  if (!batch_path_ok(B, d, F) || L.px != 3 || L.mpad != 16 * batch_mt(B)) return hipErrorInvalidValue;
  uint16_t* xp = reinterpret_cast<uint16_t*>(ws + L.xp);
  hipError_t e;
  {
    ProfScope prof("batch_topk_prep", stream);
    if (cats_unit_ok(B, d)) {
      klaunch(prep_pieces_kernel<3>, L.mpad, 256, 0, stream, x, B, d, L.mpad, norm_eps, xp);
      e = hipGetLastError();
    } else {
      e = launch_prep_frag(x, B, d, norm_eps, 3, reinterpret_cast<char*>(xp), stream);
    }
    if (e != hipSuccess) return e;
  }
  ProfScope prof("batch_topk_gate", stream);
  return launch_cats_tb<kModeAct>(B, L, stream, xp, wg, nullptr, d, F, 0.f, act, nullptr, nullptr,
                                  nullptr, nullptr, nullptr, nullptr, nullptr);
}

}  // namespace sirius
