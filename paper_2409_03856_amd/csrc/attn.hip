// Attention over the KV cache shared by the sparse and the full model, with the full model's
// direct rewrite (Algorithm 1; Sec. 4, how to correct), on gfx950.
//
// A call carries n tokens per batch entry at positions p .. p + n - 1 (p = cache_pos[b]): their
// keys and values (k_new, v_new) replace the cache rows there, and token i attends causally to
// rows 0 .. p + i. n = 1 is the sparse model's decode step, n = kernel size the full model's
// verification pass over the drafted chunk. Query head h reads key/value head h / G
// (G = H / Hkv); the G x n query rows that share a key/value head are processed together, so
// every key and value row is read once per call and 64 query rows.
//
//  attn_partial_kernel  grid (split, key/value head x row group, batch), four waves. The visible
//                       rows of a batch entry are cut on the device into equal chunks (the
//                       position lives there), so every split works whatever the cache's
//                       capacity. Both products run on MFMA in fp32 precision: the scaled query
//                       and the probabilities are split into three bf16 pieces that hold every
//                       bit, keys and values are bf16 already. Scores are formed as K Q^T, whose
//                       result layout (a lane holds one query row and 4 positions of each tile)
//                       is the B operand of V^T P^T when its K slots are numbered accordingly:
//                       probabilities never leave their registers, and the running max, sum and
//                       rescaling are per lane. QW of the waves' groups take 16 query rows each,
//                       the 4 / QW others split the positions of a tile and are merged in order at
//                       the end. Keys are staged row by row, values transposed (four positions
//                       of a column as one 8-byte store, swizzled), through registers one tile
//                       ahead. The row-group-0 workgroup also writes the new rows into the cache:
//                       each is written by exactly one workgroup and never read back in the call.
//                       With one split the kernel writes the normalised output itself.
//  attn_combine_kernel  one workgroup per query row: the chunks' (max, sum) and outputs
//                       requested together, the weights exp(m_c - M) (one chunk per thread),
//                       then each thread sums its output column over the chunks in order.
//  kv_rollback_kernel   cache_pos[b] += min(accept_len[b] + 1, n).
//
// Bound: HBM for one token (2 L Hkv hd 2 bytes) and launch latency at short contexts; at 16 tokens
// of 4 heads per key/value head the matrix work (12 n G L hd flops with the pieces; the matrix units
// are busy for 31 % of the time) and the exponentials weigh as much as the bytes. Llama-3-8B heads,
// one token over 2048 rows: 7.8 us and 3.9 for the merge (12.0 + 4.7 with fp32 vector products and
// chunks by capacity); 16 sequences of one token over 1500-3000 rows 31 + 4 us (85 + 6); 8 sequences
// of 16 tokens over 3500-7000 rows 65 + 7 us (345 + 53). The high pieces' sums of a score are kept
// apart from the rest: 2.1e-7 off 64 bits (2.3e-7 before; 3.0e-7 in one chain).
#include <float.h>
#include <math.h>

#include "common.h"
#include "kernels.h"
#include "profile.h"
#include "ring.h"

namespace sirius {
namespace {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8_t;
typedef __attribute__((__vector_size__(4 * sizeof(float)))) float floatx4_t;

constexpr int kAttnThreads = 256;
constexpr int kMaxHd = 128;
constexpr int kMaxRowsWg = 64;            // query rows per workgroup
// chunks per call at most: the merge takes them in one load batch. One key/value head then runs on 64
// workgroups: 13.9 us over 16000 rows, 27.9 over 65000, 45.7 over 131000 (31, 48 and 69 with the vector
// kernels on up to 256).
constexpr int kMaxSplits = 64;
constexpr int kTargetWgs = 512;           // workgroups of the partial kernel
constexpr int kDirectMax = 256;           // caches up to this many rows: one chunk, no combine

// The high halves of two floats as a pair of bf16 (a in the low half).
__device__ __forceinline__ uint32_t high_halves(float a, float b) {
  return __builtin_amdgcn_perm(__float_as_uint(b), __float_as_uint(a), 0x07060302u);
}
// x less its truncation to bf16, exact; 0 where nothing is left (infinities too).
__device__ __forceinline__ float rest(float x) {
  const float h = __uint_as_float(__float_as_uint(x) & 0xffff0000u);
  return h == x ? 0.f : x - h;
}

// x less its truncation to bf16 for a finite x.
__device__ __forceinline__ float rest_finite(float x) {
  return x - __uint_as_float(__float_as_uint(x) & 0xffff0000u);
}

// e^x for x <= 0 to about one ulp: the hardware exp2 of the rounded x log2(e), times the first
// order of what the rounding left off. Below -200 (a hidden position's -inf) 0; a NaN stays one.
__device__ __forceinline__ float exp_neg(float x) {
  constexpr float kHi = 1.44269502162933349609375f, kLo = 1.9259629911e-8f, kLn2 = 0.693147180559945f;
  x = __builtin_elementwise_maximum(x, -200.f);
  const float t = x * kHi;
  const float d = fmaf(x, kLo, fmaf(x, kHi, -t));
  return __builtin_amdgcn_exp2f(t) * fmaf(d, kLn2, 1.f);
}

// One query row over positions c0 .. last of a chunk in fp32 products: scores whose value is NaN and
// hidden positions weigh nothing. Keys and values lie at offsets cofs (cache) and nofs (new rows,
// positions from p on), rs apart, in 16-byte units. Writes the output over the sum to dst, or with
// pm set the output, the maximum and the sum of the chunk.
__device__ __noinline__ void whole_row(const float* __restrict__ q, float scale, const uint4* __restrict__ k_cache,
                          const uint4* __restrict__ v_cache, const uint4* __restrict__ k_new,
                          const uint4* __restrict__ v_new, size_t cofs, size_t nofs, size_t rs, int hd, int c0,
                          int last, int p, float* __restrict__ dst, float* __restrict__ pm, float* __restrict__ pl) {
  const int lane = threadIdx.x & (kWave - 1);
  auto row = [&](const uint4* cache, const uint4* fresh, int pos) {
    return pos < p ? cache + cofs + pos * rs : fresh + nofs + (pos - p) * rs;
  };
  auto score = [&](int pos) {
    const uint4* k = row(k_cache, k_new, pos);
    float s = 0.f;
    for (int c = 0; c < hd >> 3; ++c) {
      __attribute__((aligned(16))) float x[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) x[e] = q[8 * c + e] * scale;
      s = dot8(k[c], x, s);
    }
    return s;
  };
  float m = -INFINITY;
  for (int pos = c0 + lane; pos <= last; pos += kWave) m = fmaxf(m, score(pos));
  for (int k = 1; k < kWave; k <<= 1) m = fmaxf(m, __shfl_xor(m, k, kWave));
  float l = 0.f, o0 = 0.f, o1 = 0.f;  // columns lane and lane + 64
  for (int base = c0; base <= last; base += kWave) {
    const float s = base + lane <= last ? score(base + lane) : -INFINITY;
    const float w = s > -INFINITY ? expf(s - m) : 0.f;
    l += w;
    for (int j = 0; j < min(kWave, last + 1 - base); ++j) {
      const uint16_t* v = reinterpret_cast<const uint16_t*>(row(v_cache, v_new, base + j));
      const float wj = __shfl(w, j, kWave);
      if (lane < hd) o0 = fmaf(wj, bf16_lo(v[lane]), o0);
      if (lane + kWave < hd) o1 = fmaf(wj, bf16_lo(v[lane + kWave]), o1);
    }
  }
  l = wave_sum(l);
  const float d = pm != nullptr ? 1.f : l;
  if (lane < hd) dst[lane] = o0 / d;
  if (lane + kWave < hd) dst[lane + kWave] = o1 / d;
  if (pm != nullptr && lane == 0) {
    *pm = m;
    *pl = l;
  }
}

// KS: 32-wide steps of the head dimension (2: hd <= 64, 4: hd <= 128). QW: 16-row query tiles
// (1, 2 or 4), one per wave group; the 4 / QW waves of a group split a tile's positions. NB: 32-position
// blocks per wave and tile.
template <int KS, int QW, int NB>
__global__ __launch_bounds__(kAttnThreads, 2) void attn_partial_kernel(
    const float* __restrict__ q, const uint4* __restrict__ k_new, const uint4* __restrict__ v_new,
    uint4* __restrict__ k_cache, uint4* __restrict__ v_cache, const int32_t* __restrict__ cache_pos,
    int n, int H, int Hkv, int hd, int Lmax, int rgroups, int R, float scale,
    float* __restrict__ pm, float* __restrict__ pl, float* __restrict__ po,
    float* __restrict__ out) {
  constexpr int PW = 4 / QW;
  constexpr int TP = PW * NB * 32;              // positions per tile
  constexpr int kHd = KS * 32;                  // padded head dimension
  constexpr int kC = KS * 4;                    // 16-byte chunks of a padded row
  constexpr int kKPitch = kHd * 2 + 16;         // the 16 rows of an operand read: all banks
  constexpr int kVCh = TP / 8;                  // 16-byte chunks of a transposed value row
  constexpr int kVOfs = TP * kKPitch;
  constexpr int kKLoads = TP * kC / kAttnThreads;
  constexpr int kVTasks = TP / 4 * kC / kAttnThreads;  // four positions x 8 columns each
  constexpr int kQBytes = QW * 16 * kC * 3 * 16;
  constexpr int kKVBytes = kVOfs + kHd * TP * 2;
  constexpr int kRed = PW > 1 ? 4 * 16 * kHd * 4 : 0;
  constexpr int kLds = kQBytes > kKVBytes ? (kQBytes > kRed ? kQBytes : kRed) : (kKVBytes > kRed ? kKVBytes : kRed);
  static_assert(TP * kC % kAttnThreads == 0 && TP / 4 * kC % kAttnThreads == 0, "whole loads");
  static_assert(kVCh == 8 || kVCh == 16, "value swizzle");
  __shared__ __attribute__((aligned(16))) unsigned char lds[kLds];
  __shared__ float s_m[4][16], s_l[4][16];
  __shared__ int s_nan[4];
  const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid >> 6;
  const int fr = lane & 15, g = lane >> 4;
  const int split = blockIdx.x, nsplit = gridDim.x;
  const int kvh = blockIdx.y / rgroups, rg = blockIdx.y % rgroups, b = blockIdx.z;
  const int G = H / Hkv, hd8 = hd >> 3;
  const int r0 = rg * kMaxRowsWg, nr = min(16 * QW, R - r0);
  const size_t rowbase = ((size_t)b * Hkv + kvh) * R + r0;  // partial row index of row r0
  auto q_row = [&](int r) {  // row r0 + r of the group: token i, head h
    const int rr = r0 + r, i = rr / G, h = kvh * G + (rr - i * G);
    return (((size_t)b * n + i) * H + h) * hd;
  };
  const int p = cache_pos[b];
  const bool valid = p >= 0 && p + n <= Lmax;
  const int L = p + n;
  // the entry's rows in nsplit equal chunks of whole 32-position blocks
  const int chunk = valid ? ((L + nsplit - 1) / nsplit + 31) & ~31 : 32;
  const int c0 = split * chunk, c1 = min(c0 + chunk, L);

  if (!valid || c0 >= L) {  // nothing visible in this chunk (or a position outside the cache)
    if (out != nullptr) {  // what the merge of empty chunks gives: 0 / 0
      for (int e = tid; e < nr * hd; e += kAttnThreads) out[q_row(e / hd) + e % hd] = __builtin_nanf("");
      return;
    }
    if (tid < nr) {
      pm[(rowbase + tid) * nsplit + split] = -INFINITY;
      pl[(rowbase + tid) * nsplit + split] = 0.f;
    }
    return;
  }
  // ---- loads of one tile: keys and values from the cache below p, the new rows from p on, zero
  // past the chunk. K: 16-byte chunk tid % kC of row tid / kC + ..; V: chunk of four rows.
  const int lc = tid % kC, lr = tid / kC;
  const bool col = lc < hd8;
  const size_t rs = (size_t)Hkv * hd8;  // 16-byte units between positions
  const size_t cbase = (size_t)b * Lmax * rs + (size_t)kvh * hd8 + lc;
  const size_t nbase = (size_t)b * n * rs + (size_t)kvh * hd8 + lc;
  uint4 kw[kKLoads], vw[kVTasks][4];
  auto fetch = [&](const uint4* cache, const uint4* fresh, int pos) {
    if (!col || pos >= c1) return make_uint4(0u, 0u, 0u, 0u);
    return pos < p ? cache[cbase + pos * rs] : fresh[nbase + (pos - p) * rs];
  };
  auto load_tile = [&](int t0) {
#pragma unroll
    for (int u = 0; u < kKLoads; ++u) kw[u] = fetch(k_cache, k_new, t0 + lr + u * (kAttnThreads / kC));
#pragma unroll
    for (int u = 0; u < kVTasks; ++u)
#pragma unroll
      for (int j = 0; j < 4; ++j)
        vw[u][j] = fetch(v_cache, v_new, t0 + 4 * (lr + u * (kAttnThreads / kC)) + j);
  };
  auto v_at = [&](int c, int chunk16) {  // byte offset of 16-byte chunk chunk16 of value column c
    const int f = kVCh == 16 ? ((c >> 3) ^ c) & 15 : ((c >> 3) ^ (c >> 1)) & 7;
    return kVOfs + c * (TP * 2) + 16 * (chunk16 ^ f);
  };
  auto store_tile = [&]() {
#pragma unroll
    for (int u = 0; u < kKLoads; ++u)
      *reinterpret_cast<uint4*>(lds + (lr + u * (kAttnThreads / kC)) * kKPitch + 16 * lc) = kw[u];
#pragma unroll
    for (int u = 0; u < kVTasks; ++u) {
      // positions 4 qd .. 4 qd + 3 of a 32-position block: K slots 8 (qd & 3) + 4 (qd >> 2 & 1) ..
      const int qd = lr + u * (kAttnThreads / kC);
      const int ch = (qd >> 3) * 4 + (qd & 3), half = (qd >> 2) & 1;
      const uint32_t* a = &vw[u][0].x;
      const uint32_t* bq = &vw[u][1].x;
      const uint32_t* cq = &vw[u][2].x;
      const uint32_t* dq = &vw[u][3].x;
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const uint32_t sel = (e & 1) ? 0x07060302u : 0x05040100u;
        const uint2 w = make_uint2(__builtin_amdgcn_perm(bq[e >> 1], a[e >> 1], sel),
                                   __builtin_amdgcn_perm(dq[e >> 1], cq[e >> 1], sel));
        *reinterpret_cast<uint2*>(lds + v_at(8 * lc + e, ch) + 8 * half) = w;
      }
    }
  };
  load_tile(c0);
  // ---- the direct rewrite: the new rows of this chunk go into the cache
  if (rg == 0) {
    const int w0 = max(c0, p), ncw = (c1 - w0) * hd8;
    for (int e = tid; e < ncw; e += kAttnThreads) {
      const int j = e / hd8, c = e - j * hd8, pos = w0 + j;
      const size_t src = ((size_t)b * n + (pos - p)) * rs + (size_t)kvh * hd8 + c;
      const size_t dst = ((size_t)b * Lmax + pos) * rs + (size_t)kvh * hd8 + c;
      k_cache[dst] = k_new[src];
      v_cache[dst] = v_new[src];
    }
  }
  // ---- query rows, scaled, as three pieces in operand order [tile][step][piece][lane], then to
  // registers; rows past the group's and columns past hd are zero
  {
    uint4* s_q = reinterpret_cast<uint4*>(lds);
#pragma unroll
    for (int u = 0; u < QW * 16 * kC / kAttnThreads + (QW * 16 * kC % kAttnThreads != 0); ++u) {
      const int e = tid + u * kAttnThreads, r = e / kC, c = e % kC;
      if (r < 16 * QW) {
        float v[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
        if (r < nr && c < hd8) {
          const float4* src = reinterpret_cast<const float4*>(q + q_row(r)) + 2 * c;
          const float4 x = src[0], y = src[1];
          v[0] = x.x * scale; v[1] = x.y * scale; v[2] = x.z * scale; v[3] = x.w * scale;
          v[4] = y.x * scale; v[5] = y.y * scale; v[6] = y.z * scale; v[7] = y.w * scale;
        }
#pragma unroll
        for (int pc = 0; pc < 3; ++pc) {
          s_q[(((r >> 4) * KS + (c >> 2)) * 3 + pc) * kWave + 16 * (c & 3) + (r & 15)] =
              make_uint4(high_halves(v[0], v[1]), high_halves(v[2], v[3]), high_halves(v[4], v[5]),
                         high_halves(v[6], v[7]));
#pragma unroll
          for (int e2 = 0; e2 < 8; ++e2) v[e2] = rest(v[e2]);
        }
      }
    }
  }
  __syncthreads();
  const int qt = wave / PW, pw = wave % PW;
  bf16x8_t qf[KS][3];
#pragma unroll
  for (int i = 0; i < KS; ++i)
#pragma unroll
    for (int pc = 0; pc < 3; ++pc)
      qf[i][pc] = *reinterpret_cast<const bf16x8_t*>(lds + ((((qt * KS + i) * 3 + pc) * kWave) + lane) * 16);
  const int row = 16 * qt + fr;                                 // this lane's query row
  const int lim = row < nr ? p + (r0 + row) / G : -1;           // its last visible position
  float m = -FLT_MAX, l = 0.f;  // finite before the first visible position: -inf less it is no NaN
  floatx4_t o[2 * KS];  // columns 16 t + 4 g + e of the row
#pragma unroll
  for (int t = 0; t < 2 * KS; ++t) o[t] = floatx4_t{0.f, 0.f, 0.f, 0.f};
  ring_barrier();  // the query pieces are read: the tile buffers take their place

  for (int t0 = c0; t0 < c1; t0 += TP) {
    store_tile();
    ring_barrier();
    if (t0 + TP < c1) load_tile(t0 + TP);
    // ---- scores: lane holds positions 16 t + 4 g + e of its blocks
    floatx4_t s[NB][2];
#pragma unroll
    for (int nb = 0; nb < NB; ++nb)
#pragma unroll
      for (int t = 0; t < 2; ++t) {
        const int j = (pw * NB + nb) * 32 + 16 * t;
        floatx4_t a = floatx4_t{0.f, 0.f, 0.f, 0.f}, low = a;
#pragma unroll
        for (int i = 0; i < KS; ++i) {
          const bf16x8_t kf = *reinterpret_cast<const bf16x8_t*>(lds + (j + fr) * kKPitch + 64 * i + 16 * g);
#pragma unroll
          for (int pc = 2; pc > 0; --pc)
            low = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf, qf[i][pc], low, 0, 0, 0);
          a = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf, qf[i][0], a, 0, 0, 0);
        }
        s[nb][t] = a + low;
      }
    if (t0 + TP > min(c1, p + 1)) {  // uniform: a tile with hidden positions or past the chunk
#pragma unroll
      for (int nb = 0; nb < NB; ++nb)
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const int pos = t0 + (pw * NB + nb) * 32 + 16 * t + 4 * g + e;
            if (pos > lim || pos >= c1) s[nb][t][e] = -INFINITY;
          }
    }
    // ---- online softmax of the row
    float mx = -INFINITY;
#pragma unroll
    for (int nb = 0; nb < NB; ++nb)
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int e = 0; e < 4; ++e) mx = fmaxf(mx, s[nb][t][e]);
    mx = fmaxf(mx, __shfl_xor(mx, 16, kWave));
    mx = fmaxf(mx, __shfl_xor(mx, 32, kWave));
    const float m_new = fmaxf(m, mx);
    const float alpha = exp_neg(m - m_new);
    m = m_new;
    l *= alpha;
#pragma unroll
    for (int t = 0; t < 2 * KS; ++t) o[t] *= alpha;
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) {
      float pr[8];
      float sum = 0.f;
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const float w = exp_neg(s[nb][t][e] - m_new);
          pr[4 * t + e] = w;
          sum += w;
        }
      l += sum;
      // ---- O^T += V^T P^T: the probabilities' pieces are the B operand as they are
      bf16x8_t pf[3];
#pragma unroll
      for (int pc = 0; pc < 3; ++pc) {
        const uint4 w = make_uint4(high_halves(pr[0], pr[1]), high_halves(pr[2], pr[3]),
                                   high_halves(pr[4], pr[5]), high_halves(pr[6], pr[7]));
        pf[pc] = __builtin_bit_cast(bf16x8_t, w);
#pragma unroll
        for (int e = 0; e < 8; ++e) pr[e] = rest_finite(pr[e]);
      }
#pragma unroll
      for (int t = 0; t < 2 * KS; ++t) {
        const bf16x8_t vf = *reinterpret_cast<const bf16x8_t*>(lds + v_at(16 * t + fr, (pw * NB + nb) * 4 + g));
#pragma unroll
        for (int pc = 0; pc < 3; ++pc) o[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vf, pf[pc], o[t], 0, 0, 0);
      }
    }
    ring_barrier();  // every wave is done with the tile
  }
  // ---- this chunk's partial: max, sum and the unnormalised output per row (with one chunk, the
  // output itself: the unnormalised output over the sum, as the merge computes it)
  l += __shfl_xor(l, 16, kWave);
  l += __shfl_xor(l, 32, kWave);
  // an infinite key or value times a zero piece, or times pieces of both signs, is NaN where the
  // product is an infinity: then the chunk again, a wave per query row, from whole values
  floatx4_t chk = floatx4_t{l, 0.f, 0.f, 0.f};
#pragma unroll
  for (int t = 0; t < 2 * KS; ++t) chk += o[t];
  const float c1s = (chk[0] + chk[1]) + (chk[2] + chk[3]);
  const bool nan = __ballot(c1s != c1s) != 0;
  if (!(l > 0.f)) m = -INFINITY;  // nothing visible
  auto whole = [&](int r) {
    const size_t at = (rowbase + r) * nsplit + split;
    whole_row(q + q_row(r), scale, k_cache, v_cache, k_new, v_new, (size_t)b * Lmax * rs + (size_t)kvh * hd8,
              (size_t)b * n * rs + (size_t)kvh * hd8, rs, hd, c0, min(c1 - 1, p + (r0 + r) / G), p,
              out != nullptr ? out + q_row(r) : po + at * hd, out != nullptr ? nullptr : pm + at, pl + at);
  };
  if constexpr (PW == 1) {
    if (__builtin_expect(nan, 0)) {
      for (int r = 16 * qt; r < min(16 * qt + 16, nr); ++r) whole(r);
      return;
    }
    if (row < nr) {
      float* dst = out != nullptr ? out + q_row(row) : po + ((rowbase + row) * nsplit + split) * hd;
#pragma unroll
      for (int t = 0; t < 2 * KS; ++t) {
        const int c = 16 * t + 4 * g;
        if (c < hd) {
          const floatx4_t v = out != nullptr ? o[t] / l : o[t];
          *reinterpret_cast<float4*>(dst + c) = make_float4(v[0], v[1], v[2], v[3]);
        }
      }
      if (out == nullptr && g == 0) {
        pm[(rowbase + row) * nsplit + split] = m;
        pl[(rowbase + row) * nsplit + split] = l;
      }
    }
  } else {
    // the PW position groups of each query tile, merged in order through LDS
    if (lane == 0) s_nan[wave] = nan;
    if (g == 0) {
      s_m[wave][fr] = m;
      s_l[wave][fr] = l;
    }
    __syncthreads();
    if (__builtin_expect(s_nan[0] | s_nan[1] | s_nan[2] | s_nan[3], 0)) {  // uniform
      for (int r = wave; r < nr; r += kAttnThreads / kWave) whole(r);
      return;
    }
    float M = -INFINITY;
#pragma unroll
    for (int w = 0; w < PW; ++w) M = fmaxf(M, s_m[qt * PW + w][fr]);
    const float f = m > -INFINITY ? expf(m - M) : 0.f;
    float4* s_o = reinterpret_cast<float4*>(lds);  // [wave][row][kHd / 4], float4s swizzled by row
#pragma unroll
    for (int t = 0; t < 2 * KS; ++t)
      s_o[(wave * 16 + fr) * (kHd / 4) + ((4 * t + g) ^ (fr & 7))] =
          make_float4(o[t][0] * f, o[t][1] * f, o[t][2] * f, o[t][3] * f);
    __syncthreads();
    for (int e = tid; e < nr * (kHd / 4); e += kAttnThreads) {
      const int r = e / (kHd / 4), c4 = e % (kHd / 4);
      if (4 * c4 >= hd) continue;
      const int w0 = (r >> 4) * PW, rr = r & 15;
      float Mr = -INFINITY;
#pragma unroll
      for (int w = 0; w < PW; ++w) Mr = fmaxf(Mr, s_m[w0 + w][rr]);
      float4 t = make_float4(0.f, 0.f, 0.f, 0.f);
      float lt = 0.f;
#pragma unroll
      for (int w = 0; w < PW; ++w) {
        const float4 v = s_o[((w0 + w) * 16 + rr) * (kHd / 4) + (c4 ^ (rr & 7))];
        t.x += v.x; t.y += v.y; t.z += v.z; t.w += v.w;
        const float mw = s_m[w0 + w][rr];
        lt += mw > -INFINITY ? s_l[w0 + w][rr] * expf(mw - Mr) : 0.f;
      }
      if (out != nullptr) {
        *reinterpret_cast<float4*>(out + q_row(r) + 4 * c4) = make_float4(t.x / lt, t.y / lt, t.z / lt, t.w / lt);
      } else {
        *reinterpret_cast<float4*>(po + ((rowbase + r) * nsplit + split) * hd + 4 * c4) = t;
        if (c4 == 0) {
          pm[(rowbase + r) * nsplit + split] = Mr;
          pl[(rowbase + r) * nsplit + split] = lt;
        }
      }
    }
  }
}

// One workgroup (hd threads) per query row. Every thread requests its chunk's (max, sum) and
// the chunk outputs of its column together, so the row costs about one memory round trip; the
// maximum over the chunks, the weights exp(m_c - M) (one chunk per thread, LDS) and the
// denominator follow, then each thread sums its output column over the chunks in order. Chunks with
// no visible position never write their outputs: those are read but replaced by 0 (a select, so
// whatever the buffer holds there cannot reach the sum). NB: chunks at most; unrolled guards for
// more than there are cost more than they save.
template <int NB>
__device__ __forceinline__ void combine_row(int n, int H, int Hkv, int hd, int R, int nsplit,
                                            const float* __restrict__ pm,
                                            const float* __restrict__ pl,
                                            const float* __restrict__ po, float* __restrict__ out,
                                            float* s_w, float* s_red) {
  const int row = blockIdx.x;  // (b, kvh, r)
  const int r = row % R, bk = row / R, kvh = bk % Hkv, b = bk / Hkv;
  const int G = H / Hkv, i = r / G, h = kvh * G + (r - i * G);
  const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid >> 6;
  const float* o = po + (size_t)row * nsplit * hd + (tid < hd ? tid : 0);
  const float mv = tid < nsplit ? pm[(size_t)row * nsplit + tid] : -INFINITY;
  const float lv = tid < nsplit ? pl[(size_t)row * nsplit + tid] : 0.f;
  float ov[NB];
#pragma unroll
  for (int u = 0; u < NB; ++u) ov[u] = u < nsplit ? o[(size_t)u * hd] : 0.f;

  static_assert(kMaxSplits <= kWave, "the chunks' sums and weights are the first wave's");
  if (wave == 0) {
    float M = mv;
    for (int k = 1; k < kWave; k <<= 1) M = fmaxf(M, __shfl_xor(M, k, kWave));
    const float w = (mv > -INFINITY) ? expf(mv - M) : 0.f;
    float den = lv * w;
    for (int k = 1; k < kWave; k <<= 1) den += __shfl_xor(den, k, kWave);
    s_w[lane] = w;
    if (lane == 0) s_red[0] = den;
  }
  __syncthreads();
  const float den = s_red[0];
  float num = 0.f;
#pragma unroll
  for (int u = 0; u < NB; ++u) {
    if (u < nsplit) {
      const float w = s_w[u];
      num = fmaf(w > 0.f ? ov[u] : 0.f, w, num);
    }
  }
  if (tid < hd) out[(((size_t)b * n + i) * H + h) * hd + tid] = num / den;
}

__global__ __launch_bounds__(kMaxHd) void attn_combine_kernel(
    int n, int H, int Hkv, int hd, int R, int nsplit, const float* __restrict__ pm,
    const float* __restrict__ pl, const float* __restrict__ po, float* __restrict__ out) {
  __shared__ float s_w[kWave], s_red[1];
  if (nsplit <= 8)
    combine_row<8>(n, H, Hkv, hd, R, nsplit, pm, pl, po, out, s_w, s_red);
  else if (nsplit <= 32)
    combine_row<32>(n, H, Hkv, hd, R, nsplit, pm, pl, po, out, s_w, s_red);
  else
    combine_row<kMaxSplits>(n, H, Hkv, hd, R, nsplit, pm, pl, po, out, s_w, s_red);
}

__global__ void kv_rollback_kernel(int32_t* __restrict__ cache_pos,
                                   const int32_t* __restrict__ accept_len, int B, int n) {
  const int b = blockIdx.x * blockDim.x + threadIdx.x;
  if (b < B) {
    const int a = accept_len[b];
    cache_pos[b] += min(max(a, 0) + 1, n);
  }
}

}  // namespace

AttnLayout attn_layout(int B, int n, int H, int Hkv, int hd, int Lmax) {
  AttnLayout L{};
  const int R = (H / Hkv) * n;
  L.rgroups = ceil_div(R, kMaxRowsWg);
  const long wgs = (long)std::max(B, 1) * Hkv * L.rgroups;
  // Two workgroups per CU (512 in all): with 256, 1024 and 2048 the 16-token chunks of 8 sequences
  // took 95, 82 and 99 us against 78, 16 decoded tokens 41, 38 and 44 against 36; and no more chunks
  // than a full cache has tiles.
  const int tile = R <= 16 || hd <= 64 ? 128 : 64;
  L.nsplit = Lmax <= kDirectMax ? 1
                                : (int)std::max(1l, std::min<long>({(kTargetWgs + wgs - 1) / wgs,
                                                                    (long)ceil_div(Lmax, tile), (long)kMaxSplits}));
  // Room for rows * nsplit partials, by a bound that grows with every size (nsplit itself falls as the
  // batch grows), so that a workspace of the largest call serves every smaller one.
  const size_t rows = (size_t)B * Hkv * R;
  const size_t parts = Lmax <= kDirectMax ? rows
                                          : std::min(rows * std::min(kMaxSplits, ceil_div(Lmax, 64)),
                                                     rows + (size_t)(kTargetWgs - 1) * std::min(R, kMaxRowsWg));
  Carve c;
  L.pm = c.take(parts * sizeof(float));
  L.pl = c.take(parts * sizeof(float));
  L.po = c.take(parts * hd * sizeof(float));
  L.total = c.off;
  return L;
}

hipError_t launch_attn_kv(const float* q, const uint16_t* k_new, const uint16_t* v_new,
                          uint16_t* k_cache, uint16_t* v_cache, const int32_t* cache_pos, int B,
                          int n, int H, int Hkv, int hd, int Lmax, float* out, char* ws,
                          const AttnLayout& L, hipStream_t stream) {
  if (hd > kMaxHd || (hd & 7) != 0 || H % Hkv != 0) return hipErrorInvalidValue;
  const int R = (H / Hkv) * n;
  float* pm = reinterpret_cast<float*>(ws + L.pm);
  float* pl = reinterpret_cast<float*>(ws + L.pl);
  float* po = reinterpret_cast<float*>(ws + L.po);
  const float scale = (float)(1.0 / sqrt((double)hd));
  const dim3 grid(L.nsplit, Hkv * L.rgroups, B);
  const bool direct = L.nsplit == 1;  // the partial kernel writes the output; no merge
  {
    ProfScope prof("attn_partial", stream);
#define SIRIUS_ATTN(KS, QW, NB)                                                                       \
  klaunch(attn_partial_kernel<KS, QW, NB>, grid, kAttnThreads, 0, stream, q,                          \
          reinterpret_cast<const uint4*>(k_new), reinterpret_cast<const uint4*>(v_new),               \
          reinterpret_cast<uint4*>(k_cache), reinterpret_cast<uint4*>(v_cache), cache_pos, n, H, Hkv, \
          hd, Lmax, L.rgroups, R, scale, pm, pl, po, direct ? out : nullptr)
    if (hd <= 64) {
      if (R <= 16) SIRIUS_ATTN(2, 1, 1);
      else if (R <= 32) SIRIUS_ATTN(2, 2, 2);
      else SIRIUS_ATTN(2, 4, 4);
    } else {
      if (R <= 16) SIRIUS_ATTN(4, 1, 1);
      else if (R <= 32) SIRIUS_ATTN(4, 2, 1);
      else SIRIUS_ATTN(4, 4, 2);
    }
#undef SIRIUS_ATTN
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  if (direct) return hipSuccess;
  ProfScope prof("attn_combine", stream);
  klaunch(attn_combine_kernel, B * Hkv * R, kMaxHd, 0, stream, n, H, Hkv, hd, R, L.nsplit, pm, pl, po,
                                                          out);
  return hipGetLastError();
}

hipError_t launch_kv_rollback(int32_t* cache_pos, const int32_t* accept_len, int B, int n,
                              hipStream_t stream) {
  ProfScope prof("kv_rollback", stream);
  klaunch(kv_rollback_kernel, ceil_div(B, 256), 256, 0, stream, cache_pos, accept_len, B, n);
  return hipGetLastError();
}

}  // namespace sirius
