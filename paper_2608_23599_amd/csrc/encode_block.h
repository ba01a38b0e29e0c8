// Device encoder of one 64-token x 128-channel tensor block (section 3.2): source rows
// or a record -> the record of a lower level, by one workgroup of 256 threads.
//
// Every stored number is exact-reproducible: scales, zeros, codes, centroids and ids are
// those of fp64 arithmetic with one rounding per operation and one round-to-nearest-even
// to fp16.  The fast paths below compute in fp32 or on the matrix cores only what decides
// nothing, or what is decided with a proven margin, and take the fp64 path otherwise.
//
// Work split.  Thread (tg, a) holds tokens 4 tg .. 4 tg + 3, channels 8 a .. 8 a + 7 of
// the block in registers (tg = 4 * wavefront + lane / 16, a from the low four lane bits):
// a wavefront loads one 16-token page of rows, whole 256-byte rows per instruction, and
// holds every code of that page, so it assembles the page's packed words itself.  A
// channel's 64 tokens are spread over the four wavefronts, a token's 128 channels over
// one 16-lane row.  Demoting 32 blocks exact -> int8 takes 11 us this way, 43 us
// with the block in LDS, fp64 per element and one thread per channel (quantize_kernel has
// the prefill's figures).
#pragma once

#include "gkv_internal.h"

#pragma clang fp contract(off)

namespace gkv {
namespace enc {

typedef _Float16 h2 __attribute__((ext_vector_type(2)));
typedef _Float16 h8 __attribute__((ext_vector_type(8)));
typedef float f4 __attribute__((ext_vector_type(4)));
typedef uint32_t u4 __attribute__((ext_vector_type(4)));

constexpr int kThreads = 256;
constexpr int XS = D + 1;       // LDS row stride of fp64 rows (bank spread)
constexpr int XR = D + 8;       // LDS row stride of fp16 rows (halves; 16-byte aligned)
constexpr int kTermCols = 12;   // centroid k's fp16 terms are MFMA columns k, 4 + k, 8 + k

// Low four lane bits -> channel group: lane bits 0, 1 are the group's bits 1, 2, so that
// the lanes whose codes share a packed word lie in one quad.
__device__ __forceinline__ int lane_group(int l) {
  return ((l >> 2) & 1) | ((l & 1) << 1) | (((l >> 1) & 1) << 2) | (l & 8);
}

template <int CTRL>
__device__ __forceinline__ uint32_t dpp(uint32_t x) {
  return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, CTRL, 0xF, 0xF, true);
}
template <int CTRL>
__device__ __forceinline__ float dppf(float x) {
  return __uint_as_float(dpp<CTRL>(__float_as_uint(x)));
}
template <int CTRL>
__device__ __forceinline__ double dppd(double x) {
  const uint64_t b = __builtin_bit_cast(uint64_t, x);
  return __builtin_bit_cast(double, ((uint64_t)dpp<CTRL>((uint32_t)(b >> 32)) << 32) | dpp<CTRL>((uint32_t)b));
}
constexpr int kXor1 = 0xB1, kXor2 = 0x4E, kHalfMirror = 0x141, kMirror = 0x140;
// Combines x over the 16 lanes of a row (every lane gets the result).
template <class F>
__device__ __forceinline__ double row_all_d(double x, F op) {
  x = op(x, dppd<kXor1>(x));
  x = op(x, dppd<kXor2>(x));
  x = op(x, dppd<kHalfMirror>(x));
  return op(x, dppd<kMirror>(x));
}

__device__ __forceinline__ h2 as_h2(uint32_t x) { return __builtin_bit_cast(h2, x); }
__device__ __forceinline__ uint32_t as_u(h2 x) { return __builtin_bit_cast(uint32_t, x); }
// Inline assembly's results are not known to the compiler as vector-ALU results, so it adds
// no wait states before a DPP or permlane instruction that reads them: they pass through
// here first.
template <class T>
__device__ __forceinline__ void settle(T &a) {
  asm volatile("s_nop 4" : "+v"(a));
}
__device__ __forceinline__ void settle(uint32_t &a, uint32_t &b) { asm volatile("s_nop 4" : "+v"(a), "+v"(b)); }
__device__ __forceinline__ void settle(uint32_t (&a)[4], uint32_t (&b)[4]) {
  asm volatile("s_nop 4" : "+v"(a[0]), "+v"(a[1]), "+v"(a[2]), "+v"(a[3]), "+v"(b[0]), "+v"(b[1]), "+v"(b[2]), "+v"(b[3]));
}

// Packed fp16 minimum and maximum as one instruction: a quiet NaN operand is ignored.
// (The builtins first quiet both operands of each; here the words are quieted once.)
__device__ __forceinline__ uint32_t pk_min(uint32_t a, uint32_t b) {
  uint32_t r;
  asm("v_pk_min_f16 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
  return r;
}
__device__ __forceinline__ uint32_t pk_max(uint32_t a, uint32_t b) {
  uint32_t r;
  asm("v_pk_max_f16 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
  return r;
}
__device__ __forceinline__ uint32_t pk_quiet(uint32_t a) { return pk_max(a, a); }
template <class F>
__device__ __forceinline__ uint32_t over_kg(uint32_t x, F op) {  // over lanes l ^ 16, l ^ 32
  const auto a = __builtin_amdgcn_permlane32_swap(x, x, false, false);
  x = op(a[0], a[1]);
  const auto b = __builtin_amdgcn_permlane16_swap(x, x, false, false);
  return op(b[0], b[1]);
}

// ---------------------------------------------------------------- sources
// A thread's 4 x 8 elements: fp16 values (rows, an exact record) or the exact fp64 values
// of a decoded record.
struct HalfSrc {
  static constexpr bool kHalf = true;
  uint32_t w[4][4];  // row r, channel pair
  __device__ __forceinline__ uint16_t bits(int r, int e) const { return (uint16_t)(w[r][e >> 1] >> (16 * (e & 1))); }
  __device__ __forceinline__ float f(int r, int e) const { return (float)__builtin_bit_cast(_Float16, bits(r, e)); }
  __device__ __forceinline__ double d(int r, int e) const { return (double)f(r, e); }
  __device__ __forceinline__ double d_late(int r, int e) const {
    uint32_t x = w[r][e >> 1];
    asm volatile("" : "+v"(x));
    return (double)(float)__builtin_bit_cast(_Float16, (uint16_t)(x >> (16 * (e & 1))));
  }
  // Values derived from the words before this point are not kept for use after it (the
  // conversions are cheaper than the registers that hold 32 of them).
  __device__ __forceinline__ void fresh() {
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
      for (int i = 0; i < 4; ++i) asm volatile("" : "+v"(w[r][i]));
  }
  // x - z, rounded once (the mixed-precision form reads the fp16 half as it is)
  __device__ __forceinline__ float minus(int r, int e, float z) const {
    float o;
    if (e & 1) asm("v_fma_mix_f32 %0, %1, 1.0, -%2 op_sel:[1,0,0] op_sel_hi:[1,0,0]" : "=v"(o) : "v"(w[r][e >> 1]), "v"(z));
    else asm("v_fma_mix_f32 %0, %1, 1.0, -%2 op_sel_hi:[1,0,0]" : "=v"(o) : "v"(w[r][e >> 1]), "v"(z));
    return o;
  }
  // n + x^2, rounded once
  __device__ __forceinline__ float square_plus(int r, int e, float n) const {
    if (e & 1) asm("v_fma_mix_f32 %0, %1, %1, %0 op_sel:[1,1,0] op_sel_hi:[1,1,0]" : "+v"(n) : "v"(w[r][e >> 1]));
    else asm("v_fma_mix_f32 %0, %1, %1, %0 op_sel_hi:[1,1,0]" : "+v"(n) : "v"(w[r][e >> 1]));
    return n;
  }
};
struct WideSrc {
  static constexpr bool kHalf = false;
  double v[4][8];
  __device__ __forceinline__ void fresh() {}
  __device__ __forceinline__ double d_late(int r, int e) const { return v[r][e]; }
  __device__ __forceinline__ double d(int r, int e) const { return v[r][e]; }
};

// Where a thread stands in its block.
struct Place {
  int wave, lane, kg, a, tg;
  __device__ __forceinline__ Place() {
    wave = threadIdx.x >> 6;
    lane = threadIdx.x & 63;
    kg = lane >> 4;
    a = lane_group(lane & 15);
    tg = 4 * wave + kg;
  }
  // byte index (in chunks) of a key token row's chunk, and of a value channel's chunk
  __device__ __forceinline__ int kchunk(int r) const { return wave * 64 + (a & 3) * 16 + 4 * kg + r; }
  __device__ __forceinline__ int vchunk(int e) const { return wave * 64 + kg * 16 + 8 * (a & 1) + e; }
};

// Rows row0 .. row0 + 63 of one (b, h); rows at or beyond T read as zero.
__device__ __forceinline__ void load_rows(HalfSrc &s, const Place &pl, const uint16_t *src, int64_t T, int64_t row0) {
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int64_t row = row0 + 4 * pl.tg + r;
    u4 v = {0, 0, 0, 0};
    if (row < T) v = __builtin_nontemporal_load((const u4 *)(src + row * D + 8 * pl.a));
#pragma unroll
    for (int i = 0; i < 4; ++i) s.w[r][i] = v[i];
  }
}

constexpr uint32_t kPermLo = 0x05040100u, kPermHi = 0x07060302u;

template <int TENSOR>
__device__ __forceinline__ void load_exact(HalfSrc &s, const Place &pl, const uint8_t *rec) {
  if (TENSOR == GKV_KEYS) {
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const uint4 v = *(const uint4 *)(rec + pl.kchunk(r) * 64 + 16 * (pl.a >> 2));
      s.w[r][0] = v.x; s.w[r][1] = v.y; s.w[r][2] = v.z; s.w[r][3] = v.w;
    }
  } else {
#pragma unroll
    for (int p = 0; p < 4; ++p) {  // channels 2p, 2p + 1: words hold tokens (0, 1) and (2, 3)
      const uint2 lo = *(const uint2 *)(rec + pl.vchunk(2 * p) * 64 + 8 * (pl.a >> 1));
      const uint2 hi = *(const uint2 *)(rec + pl.vchunk(2 * p + 1) * 64 + 8 * (pl.a >> 1));
      s.w[0][p] = __builtin_amdgcn_perm(hi.x, lo.x, kPermLo);
      s.w[1][p] = __builtin_amdgcn_perm(hi.x, lo.x, kPermHi);
      s.w[2][p] = __builtin_amdgcn_perm(hi.y, lo.y, kPermLo);
      s.w[3][p] = __builtin_amdgcn_perm(hi.y, lo.y, kPermHi);
    }
  }
}

// Scale / zero entry (lane order of the record) of channel c.
template <int TENSOR>
__device__ __forceinline__ int sz_entry(int c) {
  return TENSOR == GKV_KEYS ? 32 * ((c >> 3) & 3) + 8 * (c >> 5) + (c & 7)
                            : 32 * ((c >> 2) & 3) + 4 * (c >> 4) + (c & 3);
}

__device__ __forceinline__ double h2d(uint16_t h) { return (double)(float)__builtin_bit_cast(_Float16, h); }

// The decoded values code * scale + zero of an int record (both steps exact in fp64).
template <int TENSOR, int BITS, bool PER_TOKEN>
__device__ __forceinline__ void load_codes(WideSrc &s, const Place &pl, const uint8_t *rec) {
  const uint16_t *hh = (const uint16_t *)rec;
  const uint32_t *w = (const uint32_t *)(rec + kSZBytes);
  constexpr int kPer = 32 / BITS;  // codes per word
  // keys: codes n = 8 (a >> 2) + e of row r's chunk; values: n = 4 (a >> 1) + r of channel e's
  const int n0 = TENSOR == GKV_KEYS ? 8 * (pl.a >> 2) : 4 * (pl.a >> 1);
#pragma unroll
  for (int e = 0; e < 8; ++e)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int o = TENSOR == GKV_KEYS ? e : r, ck = TENSOR == GKV_KEYS ? pl.kchunk(r) : pl.vchunk(e);
      int pos = code_pos(BITS, o);  // the place of code o, 4 + o, .. of a word, by n0
      constexpr int kStep = TENSOR == GKV_KEYS ? 8 : 4;
#pragma unroll
      for (int q = 1; q < kPer / kStep; ++q) pos = (n0 % kPer) == q * kStep ? code_pos(BITS, q * kStep + o) : pos;
      const uint32_t code = __builtin_amdgcn_ubfe(w[ck * BITS + (n0 + o) / kPer], (uint32_t)pos, BITS);
      const int g = PER_TOKEN ? 4 * pl.tg + r : sz_entry<TENSOR>(8 * pl.a + e);
      const double prod = (double)code * h2d(hh[g]);
      s.v[r][e] = prod + h2d(hh[(PER_TOKEN ? P : D) + g]);
    }
}

// The decoded values of an int, centroid or one-centroid record.
template <int TENSOR, bool PER_TOKEN>
__device__ __forceinline__ void load_decoded(WideSrc &s, const Place &pl, const uint8_t *rec, int level) {
  const uint16_t *hh = (const uint16_t *)rec;
  if (level == GKV_MEAN) {
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const double x = h2d(hh[8 * pl.a + e]);
#pragma unroll
      for (int r = 0; r < 4; ++r) s.v[r][e] = x;
    }
    return;
  }
  if (level == GKV_CENTROID) {
    const uint32_t ids = rec[KC * D * 2 + pl.tg];  // the ids of tokens 4 tg .. + 3
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int k = (ids >> (2 * r)) & 3;
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const int d = 8 * pl.a + e;
        s.v[r][e] = h2d(hh[TENSOR == GKV_KEYS ? k * D + d : vcent_index(k, d)]);
      }
    }
    return;
  }
  if (level == GKV_INT8) load_codes<TENSOR, 8, PER_TOKEN>(s, pl, rec);
  else if (level == GKV_INT4) load_codes<TENSOR, 4, PER_TOKEN>(s, pl, rec);
  else load_codes<TENSOR, 2, PER_TOKEN>(s, pl, rec);
}

// ---------------------------------------------------------------- workgroup memory
struct Groups {  // the quantizer's groups (channels, or tokens): scale, zero, 1 / scale or 0
  float s[D], z[D], inv[D];
};

template <bool HALF>
struct Shared {
  static constexpr int kXBytes = HALF ? P * XR * 2 : P * XS * 8;
  union {
    struct {
      uint8_t img[4][2048];  // packed code words of each wavefront's page
      Groups g;
      union {
        u4 rh[4][16][2];         // per wavefront and channel group: minima, maxima
        double rd[4][2][D];
      };
      union {
        u4 x0h[16];  // row 0, for the NaN rule
        double x0d[D];
      };
    } q;
    struct {
      __align__(16) uint8_t x[kXBytes];  // the block: fp16 rows of XR halves, or fp64 rows of XS
      union {
        uint16_t terms[kTermCols * XR];  // the centroids as fp16 terms, one row per MFMA column
        double dist[P * KC];
      };
      double c[KC * XS];  // centroids
      float cn[KC];       // their squared norms
      float xn[P];        // the tokens' norms
      int32_t assign[P];
    } l;
    double part[16][D];  // block-mean sums of each token group
  };
  double cmean[D];
  double cert[2][16];
  float low[2][4];
};

// ---------------------------------------------------------------- certificate
// Non-negative fp64 -> fp32 rounded towards +inf (the certificate keeps upper
// bounds): one ulp up when the nearest float lies below.
__device__ __forceinline__ float round_up_f32(double x) {
  float f = (float)x;
  if ((double)f < x) f = __builtin_bit_cast(float, __builtin_bit_cast(uint32_t, f) + 1u);
  return f;
}

// Row sums over the 16 lanes that hold a token's channels (every lane gets them).
__device__ __forceinline__ float row_sum(float x) {
  x += dppf<kXor1>(x);
  x += dppf<kXor2>(x);
  x += dppf<kHalfMirror>(x);
  return x + dppf<kMirror>(x);
}
__device__ __forceinline__ double row_sum_d(double x) {
  return row_all_d(x, [](double p, double q) { return p + q; });
}

// Largest value over the wavefront's rows (the lanes of a row agree); NaN is ignored.
__device__ __forceinline__ float wave_rows_max(float x) {
  return __uint_as_float(over_kg(__float_as_uint(x), [](uint32_t p, uint32_t q) {
    return __float_as_uint(fmaxf(__uint_as_float(p), __uint_as_float(q)));
  }));
}

// err = max_t ||x_t - x_hat_t|| (ERR) and, for values, nrm = max_t ||x_t|| over the
// block's 64 rows, fp64; xhat(r, e) is this thread's reconstruction.  Valid in thread 0.
//
// fp16 blocks screen the rows first: E[r] is this thread's part of row r's sum of
// squared errors in fp32 and slack(r, sum) bounds how far the row's fp32 sum is off.
// Only rows whose upper bound reaches the largest lower bound can hold the maximum, and
// only theirs are formed in fp64 (usually one row of 64; fp64 for every element was a
// third of the encode's instructions).  A norm's fp32 sum is within 2^-16 of it (128
// additions, the products exact).
template <int TENSOR, bool ERR, bool HALF, class S, class D2, class F>
__device__ __forceinline__ void block_cert(Shared<HALF> &sh, const Place &pl, S &s, const float (&E)[4], D2 slack,
                                           F xhat, double &err, double &nrm) {
  constexpr bool NRM = TENSOR != GKV_KEYS;
  double me = 0.0, mn = 0.0;
  if constexpr (HALF) {
    float eu[4], nu[4];  // the rows' upper bounds
    float el = -1.f, nl = -1.f;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      if (ERR) {
        const float sum = row_sum(E[r]), b = slack(r, sum);
        eu[r] = sum + b;
        el = fmaxf(el, sum - b);
      }
      if (NRM) {
        float N = 0.f;
#pragma unroll
        for (int e = 0; e < 8; ++e) N = s.square_plus(r, e, N);
        settle(N);
        N = row_sum(N);
        nu[r] = N * (1.f + 0x1p-16f);
        nl = fmaxf(nl, N * (1.f - 0x1p-16f));
      }
    }
    if (ERR) el = wave_rows_max(el);
    if (NRM) nl = wave_rows_max(nl);
    if (pl.lane == 0) {
      sh.low[0][pl.wave] = el;
      sh.low[1][pl.wave] = nl;
    }
    __syncthreads();
    el = fmaxf(fmaxf(sh.low[0][0], sh.low[0][1]), fmaxf(sh.low[0][2], sh.low[0][3]));
    nl = fmaxf(fmaxf(sh.low[1][0], sh.low[1][1]), fmaxf(sh.low[1][2], sh.low[1][3]));
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      __builtin_amdgcn_sched_barrier(0);
      s.fresh();
      if (ERR && __any(eu[r] >= el)) {
        double sum = 0.0;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          const double dx = s.d(r, e) - xhat(r, e);
          sum = __builtin_fma(dx, dx, sum);
        }
        sum = row_sum_d(sum);
        me = sum > me ? sum : me;
      }
      if (NRM && __any(nu[r] >= nl)) {
        double sum = 0.0;
#pragma unroll
        for (int e = 0; e < 8; ++e) sum = __builtin_fma(s.d(r, e), s.d(r, e), sum);
        sum = row_sum_d(sum);
        mn = sum > mn ? sum : mn;
      }
    }
  } else {
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      double sum = 0.0;
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const double dx = s.d(r, e) - xhat(r, e);
        sum = __builtin_fma(dx, dx, sum);
      }
      sum = row_sum_d(sum);
      me = sum > me ? sum : me;
    }
  }
  if ((pl.lane & 15) == 0) {
    sh.cert[0][pl.tg] = me;
    sh.cert[1][pl.tg] = mn;
  }
  __syncthreads();
  if (threadIdx.x < 16) {  // 16 lanes: one row
    const auto mx = [](double p, double q) { return p > q ? p : q; };
    if (ERR) err = __builtin_sqrt(row_all_d(sh.cert[0][threadIdx.x], mx));
    if (HALF && NRM) nrm = __builtin_sqrt(row_all_d(sh.cert[1][threadIdx.x], mx));
  }
}

// The squared errors x - x_hat of fp16 values against an fp16 reconstruction, in fp32:
// one rounding of each difference, so a row's sum is within 2^-16 of it.
template <class S, class F>
__device__ __forceinline__ void half_errors(S &s, F xhat, float (&E)[4]) {
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    E[r] = 0.f;
    if constexpr (S::kHalf) {
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const float dx = s.minus(r, e, (float)xhat(r, e));
        E[r] = fmaf(dx, dx, E[r]);
      }
    }
  }
}
__device__ __forceinline__ float half_slack(int, float sum) { return 0x1p-16f * sum; }

// ---------------------------------------------------------------- int levels
// code = rint((x - z) / s) of the fp64 quotient, clamped; s = 0 gives 0.  diff and r * s
// are multiples of 2^-24 below 2^26, so the remainder diff - r s is exact and decides the
// rounding of the real quotient; a quotient that is no half-integer lies at least 2^-41
// from one, far more than the fp64 quotient's rounding, so both round alike.  NaN gives 0.
__device__ __forceinline__ float exact_code(double diff, double s, double inv, float qmax) {
  double r = __builtin_rint(diff * inv);
  const double rem2 = 2.0 * __builtin_fma(-r, s, diff);
  const bool odd = __builtin_fabs(__builtin_fma(-2.0, __builtin_rint(0.5 * r), r)) == 1.0;
  if (rem2 > s || (rem2 == s && odd)) r += 1.0;
  else if (rem2 < -s || (rem2 == -s && odd)) r -= 1.0;
  r = __builtin_fmin(__builtin_fmax(r, 0.0), (double)qmax);
  return s != 0.0 ? (float)r : 0.f;
}

// A non-negative (or NaN) fp64 rounded once to fp16: to fp32 rounded to odd, then to fp16.
__device__ __forceinline__ uint16_t pos_f64_to_f16(double x) {
  uint32_t f = __float_as_uint((float)x);
  if ((double)__uint_as_float(f) > x) f -= 1;        // towards zero
  if ((double)__uint_as_float(f) != x) f |= 1;       // inexact: odd
  const uint16_t h = __builtin_bit_cast(uint16_t, (_Float16)__uint_as_float(f));
  return x != x ? (uint16_t)((__builtin_bit_cast(uint64_t, x) >> 48 & 0x8000u) | 0x7E00u) : h;
}

// a / b, rounded once, with y = 1 / b rounded to nearest (Markstein's correction step).
__device__ __forceinline__ double div_by(double a, double b, double y) {
  const double q = a * y;
  const double c = __builtin_fma(__builtin_fma(-q, b, a), y, q);
  return __builtin_isfinite(q) ? c : q;
}

// Group statistics -> scale, zero and 1 / scale (the minimum and maximum as the fp64
// quantizer takes them; a NaN in the group's first element makes both NaN).
template <int BITS>
__device__ __forceinline__ void group_params(Groups &g, int i, double mn, double mx, double first, uint16_t &s16,
                                             uint16_t &z16) {
  constexpr double qmax = (double)((1 << BITS) - 1);
  if (first != first) mn = mx = first;
  const double range = mx - mn;
  z16 = canon_zero(f64_to_f16(mn));
  s16 = canon_zero(pos_f64_to_f16(div_by(range, qmax, 1.0 / qmax)));
  const float s = (float)__builtin_bit_cast(_Float16, s16);
  // 1 / s to half an ulp and a little: the hardware reciprocal and one Newton step
  const float y = __builtin_amdgcn_rcpf(s);
  const float inv = fmaf(fmaf(-s, y, 1.f), y, y);
  g.s[i] = s;
  g.z[i] = (float)__builtin_bit_cast(_Float16, z16);
  g.inv[i] = s != 0.f ? (s < __builtin_inff() ? inv : 0.f * s) : 0.f;
}

// Bits of this thread's codes cr[r][e] into packed words of the wavefront's page image.
template <int TENSOR, int BITS>
__device__ __forceinline__ void pack_codes(uint8_t *img, const Place &pl, const float (&cr)[4][8]) {
  const int lam = pl.lane & 15;
  if (TENSOR == GKV_KEYS) {
    const int i = pl.a >> 2;  // codes n = 8 i .. 8 i + 7 of the chunks of rows r
    const int ck = (pl.a & 3) * 16 + 4 * pl.kg;
    if (BITS == 8) {
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        uint2 w = make_uint2(0, 0);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          w.x = __builtin_amdgcn_cvt_pk_u8_f32(cr[r][e], e, w.x);
          w.y = __builtin_amdgcn_cvt_pk_u8_f32(cr[r][4 + e], e, w.y);
        }
        *(uint2 *)(img + (ck + r) * 32 + 8 * i) = w;
      }
    } else if (BITS == 4) {
      uint32_t w[4];
#pragma unroll
      for (int r = 0; r < 4; ++r) {  // byte pairs: positions 4, 20, 12, 28 of e < 4 and 0, 16, 8, 24
        w[r] = __builtin_amdgcn_cvt_pk_u8_f32(fmaf(16.f, cr[r][0], cr[r][4]), 0, 0);
        w[r] = __builtin_amdgcn_cvt_pk_u8_f32(fmaf(16.f, cr[r][2], cr[r][6]), 1, w[r]);
        w[r] = __builtin_amdgcn_cvt_pk_u8_f32(fmaf(16.f, cr[r][1], cr[r][5]), 2, w[r]);
        w[r] = __builtin_amdgcn_cvt_pk_u8_f32(fmaf(16.f, cr[r][3], cr[r][7]), 3, w[r]);
        *(uint32_t *)(img + (ck + r) * 16 + 4 * i) = w[r];
      }
    } else {
      const bool odd = i & 1;  // codes 8 .. 15 of the word
      int pos[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) pos[e] = odd ? code_pos(2, 8 + e) : code_pos(2, e);
      uint32_t w[4];
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        w[r] = 0;
#pragma unroll
        for (int e = 0; e < 8; ++e) w[r] |= (uint32_t)cr[r][e] << pos[e];
        w[r] |= dpp<kXor2>(w[r]);  // the other half of the word: group a ^ 4
      }
#pragma unroll
      for (int q = 0; q < 2; ++q) {  // each of the two lanes writes two of the four rows
        const uint32_t lo = w[q], hi = w[2 + q];
        *(uint32_t *)(img + (ck + 2 * (int)odd + q) * 8 + 4 * (i >> 1)) = odd ? hi : lo;
      }
    }
  } else {
    const int j = pl.a >> 1;  // codes n = 4 j .. 4 j + 3 (tokens r) of the chunks of channels e
    const int ck = pl.kg * 16 + 8 * (pl.a & 1);
    if (BITS == 8) {
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        uint32_t w = 0;
#pragma unroll
        for (int r = 0; r < 4; ++r) w = __builtin_amdgcn_cvt_pk_u8_f32(cr[r][e], r, w);
        *(uint32_t *)(img + (ck + e) * 32 + 4 * j) = w;
      }
    } else {
      // tokens 0, 2 lie in the low half of the word and 1, 3 at the same places of the
      // high half: int4 at 4, 12 or 0, 8 by j & 1; int2 at 8, 14 | 6, 12 | 4, 10 | 0, 2 by j & 3
      float A, B;
      if (BITS == 4) {
        A = (j & 1) ? 1.f : 16.f;
        B = 256.f * A;
      } else {
        const int q = j & 3;
        A = q == 0 ? 256.f : (q == 1 ? 64.f : (q == 2 ? 16.f : 1.f));
        B = q == 0 ? 16384.f : (q == 1 ? 4096.f : (q == 2 ? 1024.f : 4.f));
      }
      uint32_t w[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        w[e] = (uint32_t)fmaf(B, cr[2][e], A * cr[0][e]) | ((uint32_t)fmaf(B, cr[3][e], A * cr[1][e]) << 16);
        w[e] |= dpp<kXor1>(w[e]);  // group a ^ 2: j ^ 1
        if (BITS == 2) w[e] |= dpp<kXor2>(w[e]);  // group a ^ 4: j ^ 2
      }
      if (BITS == 4) {  // the two lanes of a word write four channels each
        const bool up = lam & 1;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const uint32_t lo = w[q], hi = w[4 + q];
          *(uint32_t *)(img + (ck + 4 * (int)up + q) * 16 + 4 * (j >> 1)) = up ? hi : lo;
        }
      } else {  // the four lanes two each
        const int l4 = lam & 3;
#pragma unroll
        for (int q = 0; q < 2; ++q) {
          const uint32_t w0 = w[q], w1 = w[2 + q], w2 = w[4 + q], w3 = w[6 + q];
          const uint32_t lo = (l4 & 1) ? w1 : w0, hi = (l4 & 1) ? w3 : w2;
          *(uint32_t *)(img + (ck + 2 * l4 + q) * 8 + 4 * (j >> 2)) = (l4 & 2) ? hi : lo;
        }
      }
    }
  }
}

// Scalar quantizer, one group per channel, or per token for a value block of a cache that
// groups values per token (section 3.2).
template <int TENSOR, int BITS, bool PER_TOKEN, class S>
__device__ __forceinline__ void encode_int(Shared<S::kHalf> &sh, const Place &pl, S &s, uint8_t *dst,
                                           bool cert, double &err, double &nrm) {
  constexpr float qmax = (float)((1 << BITS) - 1);
  auto &q = sh.q;
  s.fresh();
  uint16_t *sz = (uint16_t *)dst;
  // ---- the groups' minima and maxima
  if (PER_TOKEN) {
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      double mn, mx;
      const auto fmn = [](double x, double y) { return __builtin_fmin(x, y); };
      const auto fmx = [](double x, double y) { return __builtin_fmax(x, y); };
      if constexpr (S::kHalf) {
        const uint32_t w0 = pk_quiet(s.w[r][0]), w1 = pk_quiet(s.w[r][1]), w2 = pk_quiet(s.w[r][2]),
                       w3 = pk_quiet(s.w[r][3]);
        uint32_t lo = pk_min(pk_min(w0, w1), pk_min(w2, w3)), hi = pk_max(pk_max(w0, w1), pk_max(w2, w3));
        settle(lo, hi);
        lo = pk_min(lo, dpp<kXor1>(lo)); hi = pk_max(hi, dpp<kXor1>(hi));
        settle(lo, hi);
        lo = pk_min(lo, dpp<kXor2>(lo)); hi = pk_max(hi, dpp<kXor2>(hi));
        settle(lo, hi);
        lo = pk_min(lo, dpp<kHalfMirror>(lo)); hi = pk_max(hi, dpp<kHalfMirror>(hi));
        settle(lo, hi);
        lo = pk_min(lo, dpp<kMirror>(lo)); hi = pk_max(hi, dpp<kMirror>(hi));
        mn = fmn(h2d((uint16_t)lo), h2d((uint16_t)(lo >> 16)));
        mx = fmx(h2d((uint16_t)hi), h2d((uint16_t)(hi >> 16)));
      } else {
        mn = mx = s.v[r][0];
#pragma unroll
        for (int e = 1; e < 8; ++e) {
          mn = fmn(mn, s.v[r][e]);
          mx = fmx(mx, s.v[r][e]);
        }
        mn = row_all_d(mn, fmn);
        mx = row_all_d(mx, fmx);
      }
      if ((pl.lane & 15) == 0) {  // channel group 0: holds the token's channel 0
        uint16_t s16, z16;
        const int t = 4 * pl.tg + r;
        group_params<BITS>(q.g, t, mn, mx, s.d(r, 0), s16, z16);
        sz[t] = s16;  // scale[64], zero[64] in token order, then zeros
        sz[P + t] = z16;
      }
    }
    if (threadIdx.x < P) ((uint32_t *)(sz + 2 * P))[threadIdx.x] = 0;
    __syncthreads();
  } else {
    if constexpr (S::kHalf) {
      uint32_t l4[4], h4[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const uint32_t w0 = pk_quiet(s.w[0][i]), w1 = pk_quiet(s.w[1][i]), w2 = pk_quiet(s.w[2][i]),
                       w3 = pk_quiet(s.w[3][i]);
        l4[i] = pk_min(pk_min(w0, w1), pk_min(w2, w3));
        h4[i] = pk_max(pk_max(w0, w1), pk_max(w2, w3));
      }
      settle(l4, h4);
#pragma unroll
      for (int i = 0; i < 4; ++i) {  // lanes l ^ 32
        const auto x = __builtin_amdgcn_permlane32_swap(l4[i], l4[i], false, false);
        const auto y = __builtin_amdgcn_permlane32_swap(h4[i], h4[i], false, false);
        l4[i] = pk_min(x[0], x[1]);
        h4[i] = pk_max(y[0], y[1]);
      }
      settle(l4, h4);
      u4 lo, hi;
#pragma unroll
      for (int i = 0; i < 4; ++i) {  // lanes l ^ 16
        const auto x = __builtin_amdgcn_permlane16_swap(l4[i], l4[i], false, false);
        const auto y = __builtin_amdgcn_permlane16_swap(h4[i], h4[i], false, false);
        lo[i] = pk_min(x[0], x[1]);
        hi[i] = pk_max(y[0], y[1]);
      }
      if (pl.kg == 0) {
        q.rh[pl.wave][pl.a][0] = lo;
        q.rh[pl.wave][pl.a][1] = hi;
        if (pl.wave == 0) q.x0h[pl.a] = u4{s.w[0][0], s.w[0][1], s.w[0][2], s.w[0][3]};
      }
    } else {
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        double mn = s.v[0][e], mx = mn;
#pragma unroll
        for (int r = 1; r < 4; ++r) {
          mn = __builtin_fmin(mn, s.v[r][e]);
          mx = __builtin_fmax(mx, s.v[r][e]);
        }
#pragma unroll
        for (int o = 16; o <= 32; o <<= 1) {
          mn = __builtin_fmin(mn, __shfl_xor(mn, o));
          mx = __builtin_fmax(mx, __shfl_xor(mx, o));
        }
        if (pl.kg == 0) {
          q.rd[pl.wave][0][8 * pl.a + e] = mn;
          q.rd[pl.wave][1][8 * pl.a + e] = mx;
          if (pl.wave == 0) q.x0d[8 * pl.a + e] = s.v[0][e];
        }
      }
    }
    __syncthreads();
    if (threadIdx.x < D) {
      const int d = threadIdx.x;
      double mn, mx, first;
      if constexpr (S::kHalf) {
        const uint16_t *rh = (const uint16_t *)&q.rh[0][d >> 3][0] + (d & 7);
        _Float16 lo = __builtin_bit_cast(_Float16, rh[0]), hi = __builtin_bit_cast(_Float16, rh[8]);
#pragma unroll
        for (int w = 1; w < 4; ++w) {
          lo = __builtin_elementwise_min(lo, __builtin_bit_cast(_Float16, rh[w * 256]));
          hi = __builtin_elementwise_max(hi, __builtin_bit_cast(_Float16, rh[w * 256 + 8]));
        }
        mn = (double)(float)lo;
        mx = (double)(float)hi;
        first = h2d(((const uint16_t *)q.x0h)[d]);
      } else {
        mn = q.rd[0][0][d];
        mx = q.rd[0][1][d];
#pragma unroll
        for (int w = 1; w < 4; ++w) {
          mn = __builtin_fmin(mn, q.rd[w][0][d]);
          mx = __builtin_fmax(mx, q.rd[w][1][d]);
        }
        first = q.x0d[d];
      }
      uint16_t s16, z16;
      group_params<BITS>(q.g, d, mn, mx, first, s16, z16);
      const int en = sz_entry<TENSOR>(d);
      sz[en] = s16;
      sz[D + en] = z16;
    }
    __syncthreads();
  }
  // ---- codes
  const int gi = PER_TOKEN ? 4 * pl.tg : 8 * pl.a;  // this thread's first group
  constexpr int kG = PER_TOKEN ? 4 : 8;
  float gz[kG], gs[kG];
#pragma unroll
  for (int g = 0; g < kG; ++g) {
    gz[g] = q.g.z[gi + g];
    gs[g] = q.g.s[gi + g];
  }
  float cr[4][8], E[4] = {0.f, 0.f, 0.f, 0.f};
  const auto exact = [&](int r, int e) {
    // the group's numbers come from LDS again and the element through an opaque copy, so
    // that nothing of this rare path is computed ahead of it and held in registers
    int g = gi + (PER_TOKEN ? r : e);
    asm volatile("" : "+v"(g));
    cr[r][e] = exact_code(s.d_late(r, e) - (double)q.g.z[g], (double)q.g.s[g], (double)q.g.inv[g], qmax);
  };
  if constexpr (S::kHalf) {
    // fp32 quotient: x - z, 1 / s and their product are each within about 2^-24 of
    // theirs, so it is within (qmax + 1) 2^-22 of the quotient; a quotient further than
    // that from a half-integer rounds alike.  It lies in [0, qmax + 1/2): z is the
    // group's minimum, and a normal fp16 scale is within 2^-11 of range / qmax.  The
    // elements that have a lane in the margin take the fp64 path (exact ties are common,
    // since x lies on the fp16 grid: about every second wavefront of random data has
    // one), all elements where a group has a subnormal scale, an infinity or NaN.
    constexpr float lim = 0.5f - (qmax + 1.f) * 0x1p-22f;
    float inv[kG];
    bool plain = true;
#pragma unroll
    for (int g = 0; g < kG; ++g) {
      inv[g] = q.g.inv[gi + g];
      plain = plain & (inv[g] <= 0x1p14f);
    }
    uint32_t near = 0;  // wave-uniform: bit 4 e + r
#pragma unroll
    for (int e = 0; e < 8; ++e)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int g = PER_TOKEN ? r : e;
        const float d = s.minus(r, e, gz[g]), x = d * inv[g];
        cr[r][e] = __builtin_rintf(x);
        near |= __ballot(!(__builtin_fabsf(x - cr[r][e]) < lim)) != 0 ? 1u << (4 * e + r) : 0u;  // NaN too
        const float dx = fmaf(-cr[r][e], gs[g], d);
        E[r] = fmaf(dx, dx, E[r]);
        if (r == 3) {  // four elements at a time, their errors summed here
          asm volatile("" : "+v"(E[0]), "+v"(E[1]), "+v"(E[2]), "+v"(E[3]));
          __builtin_amdgcn_sched_barrier(0);
        }
      }
    plain = __all(plain);
    if (!plain) near = ~0u;
    if (near) {
      s.fresh();
#pragma unroll
      for (int e = 0; e < 8; ++e)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          if ((near >> (4 * e + r)) & 1u) exact(r, e);
          __builtin_amdgcn_sched_barrier(0);
        }
    }
    if (!plain) {
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        E[r] = 0.f;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          const int g = PER_TOKEN ? r : e;
          const float dx = fmaf(-cr[r][e], gs[g], s.minus(r, e, gz[g]));
          E[r] = fmaf(dx, dx, E[r]);
        }
      }
    }
  } else {
#pragma unroll
    for (int e = 0; e < 8; ++e)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        exact(r, e);
        if (r & 1) __builtin_amdgcn_sched_barrier(0);  // two elements at a time: few registers
      }
  }
  pack_codes<TENSOR, BITS>(q.img[pl.wave], pl, cr);
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");  // the page's words, written by this wavefront's lanes
  {
    const u4 *im = (const u4 *)q.img[pl.wave];
    u4 *o = (u4 *)(dst + kSZBytes + pl.wave * 256 * BITS);
    if (BITS == 8) {
      o[pl.lane] = im[pl.lane];
      o[64 + pl.lane] = im[64 + pl.lane];
    } else if (BITS == 4) {
      o[pl.lane] = im[pl.lane];
    } else if (pl.lane < 32) {
      o[pl.lane] = im[pl.lane];
    }
  }
  if (cert) {
    // A row's fp32 sum of squares E: each element's error is within 2^-24 (|e| + x - z) of
    // its own, with x - z below Q s (Q = qmax + 1), so with S = sum of s^2 over the row E
    // is within 2^-17 E + 2^-23 2 Q sqrt(E S) + 2^-48 Q^2 S of it (Cauchy; twice that and
    // more is taken); a code that the fp64 path moved has its two errors within Q 2^-21 s
    // of each other, another Q 2^-21 S.
    constexpr float Q = qmax + 1.f;
    float s2[4] = {0.f, 0.f, 0.f, 0.f};
    if constexpr (S::kHalf) {
      if (PER_TOKEN) {
#pragma unroll
        for (int r = 0; r < 4; ++r) s2[r] = (float)D * gs[r] * gs[r];
      } else {
        float t = 0.f;
#pragma unroll
        for (int e = 0; e < 8; ++e) t = fmaf(gs[e], gs[e], t);
        s2[0] = s2[1] = s2[2] = s2[3] = row_sum(t);
      }
    }
    block_cert<TENSOR, true>(
        sh, pl, s, E,
        [&](int r, float sum) {
          return fmaf(0x1p-16f, sum, fmaf(Q * 0x1p-21f, __builtin_amdgcn_sqrtf(sum * s2[r]), Q * 0x1p-20f * s2[r]));
        },
        [&](int r, int e) {
          const int g = PER_TOKEN ? r : e;
          return __builtin_fma((double)cr[r][e], (double)gs[g], (double)gz[g]);  // exact
        },
        err, nrm);
  }
}

// ---------------------------------------------------------------- exact level
template <int TENSOR>
__device__ __forceinline__ void write_exact(const Place &pl, const HalfSrc &s, uint8_t *dst) {
  if (TENSOR == GKV_KEYS) {
#pragma unroll
    for (int r = 0; r < 4; ++r)
      *(uint4 *)(dst + pl.kchunk(r) * 64 + 16 * (pl.a >> 2)) = make_uint4(s.w[r][0], s.w[r][1], s.w[r][2], s.w[r][3]);
  } else {
#pragma unroll
    for (int p = 0; p < 4; ++p)
#pragma unroll
      for (int o = 0; o < 2; ++o) {
        const uint32_t sel = o ? kPermHi : kPermLo;
        *(uint2 *)(dst + pl.vchunk(2 * p + o) * 64 + 8 * (pl.a >> 1)) =
            make_uint2(__builtin_amdgcn_perm(s.w[1][p], s.w[0][p], sel), __builtin_amdgcn_perm(s.w[3][p], s.w[2][p], sel));
      }
  }
}

// ---------------------------------------------------------------- one-centroid state
// The Lloyd iteration with one centroid converges in one update to the block mean; the
// sum of 64 fp16 (or decoded) values is exact in fp64 (all are multiples of 2^-24 below
// 2^18), so its order does not matter, then one fp16 rounding.
template <int TENSOR, class S>
__device__ __forceinline__ void encode_mean(Shared<S::kHalf> &sh, const Place &pl, S &s, uint8_t *dst,
                                            bool cert, double &err, double &nrm) {
  s.fresh();
#pragma unroll
  for (int e = 0; e < 8; ++e)
    sh.part[pl.tg][8 * pl.a + e] = (s.d(0, e) + s.d(1, e)) + (s.d(2, e) + s.d(3, e));
  __syncthreads();
  if (threadIdx.x < D) {
    double acc = sh.part[0][threadIdx.x];
#pragma unroll
    for (int i = 1; i < 16; ++i) acc = acc + sh.part[i][threadIdx.x];
    const uint16_t h = canon_zero(f64_to_f16(acc / (double)P));
    sh.cmean[threadIdx.x] = f16_to_f64(h);
    ((uint16_t *)dst)[threadIdx.x] = h;
  }
  if (cert) {
    __syncthreads();
    const auto xh = [&](int r, int e) { return sh.cmean[8 * pl.a + e]; };
    float E[4];
    half_errors(s, xh, E);
    block_cert<TENSOR, true>(sh, pl, s, E, half_slack, xh, err, nrm);
  }
}

// ---------------------------------------------------------------- centroid state
// Element (t, d) of the staged block.
template <bool HALF>
__device__ __forceinline__ double staged(const Shared<HALF> &sh, int t, int d) {
  if (HALF) return h2d(((const uint16_t *)sh.l.x)[t * XR + d]);
  return ((const double *)sh.l.x)[t * XS + d];
}

// Elements (t, 2 lane) and (t, 2 lane + 1).
template <bool HALF>
__device__ __forceinline__ double2 staged2(const Shared<HALF> &sh, int t, int lane) {
  if (HALF) {
    const uint32_t w = *(const uint32_t *)((const uint16_t *)sh.l.x + t * XR + 2 * lane);
    return make_double2(h2d((uint16_t)w), h2d((uint16_t)(w >> 16)));
  }
  const double *x = (const double *)sh.l.x + t * XS + 2 * lane;
  return make_double2(x[0], x[1]);
}

// Every token's nearest centroid from the fp64 squared distances, channel-ascending, no
// fused multiply-add, ties to the lower centroid: the definition of the ids.
template <bool HALF>
__device__ __forceinline__ void assign_exact(Shared<HALF> &sh) {
  const int t = threadIdx.x >> 2, k = threadIdx.x & 3;  // 256 threads = 64 tokens x 4
  double acc = 0.0;
#pragma unroll 8
  for (int d = 0; d < D; ++d) {
    const double diff = staged(sh, t, d) - sh.l.c[k * XS + d];
    const double sq = diff * diff;
    acc = acc + sq;
  }
  __syncthreads();  // dist shares its space with the terms
  sh.l.dist[t * KC + k] = acc;
  __syncthreads();
  if (threadIdx.x < P) {
    const int tt = threadIdx.x;
    int best = 0;
    double bd = sh.l.dist[tt * KC];
    for (int kk = 1; kk < KC; ++kk)
      if (sh.l.dist[tt * KC + kk] < bd) {
        bd = sh.l.dist[tt * KC + kk];
        best = kk;
      }
    sh.l.assign[tt] = best;
  }
  __syncthreads();
}

// Wavefront k: centroid k's fp16 terms c = hi + mid 2^-11 + lo 2^-22 (to 2^-33 |c|) and
// its squared norm, from its channels 2 lane, 2 lane + 1.
__device__ __forceinline__ void write_terms(Shared<true> &sh, const Place &pl, double c0, double c1) {
  const double c[2] = {c0, c1};
  uint16_t t[3][2];
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const _Float16 hi = (_Float16)(float)c[i];
    const double r1 = c[i] - (double)(float)hi;
    const _Float16 mid = (_Float16)((float)r1 * 0x1p11f);
    const double r2 = r1 - (double)(float)mid * 0x1p-11;
    const _Float16 lo = (_Float16)((float)r2 * 0x1p22f);
    t[0][i] = __builtin_bit_cast(uint16_t, hi);
    t[1][i] = __builtin_bit_cast(uint16_t, mid);
    t[2][i] = __builtin_bit_cast(uint16_t, lo);
  }
#pragma unroll
  for (int q = 0; q < 3; ++q)
    *(uint32_t *)(sh.l.terms + (4 * q + pl.wave) * XR + 2 * pl.lane) = (uint32_t)t[q][0] | ((uint32_t)t[q][1] << 16);
  const float f0 = (float)c0, f1 = (float)c1;
  const float n = __uint_as_float(over_kg(__float_as_uint(row_sum(fmaf(f0, f0, f1 * f1))), [](uint32_t p, uint32_t q) {
    return __float_as_uint(__uint_as_float(p) + __uint_as_float(q));
  }));
  if (pl.lane == 0) sh.l.cn[pl.wave] = n;
}

// Every token's nearest centroid, for fp16 blocks: one MFMA chain per 16-token page gives
// x . c for the three terms of the four centroids, and |c|^2 - 2 x . c orders the
// distances.  x . c is off by at most 2^-16 |x| |c| (128 products, each addition within
// 2^-23 of a partial sum below |x| |c|), twice that in a distance and four times in the gap
// of two: 2^-14 |x| |c|.  |c|^2 is off by 10 units of 2^-24 |c|^2 (two for the square of a
// centroid rounded to fp32, two for the pair, six additions over the lanes) and the
// distance's own rounding adds one: 22 units, below 2^-19 |c|^2, in the gap of two.  A gap
// between the two nearest of more than 2^-13 |x| |c| + 2^-18 max |c|^2 therefore decides as
// the fp64 distances do (fp16 subnormals enter these MFMAs as they are); a block with a
// token inside the margin takes the fp64 distances.  The second term counts for tokens
// near zero only.  Workgroup-uniform; assign is complete after it.
__device__ __forceinline__ void assign_fast(Shared<true> &sh, const Place &pl, const h8 (&xa)[4]) {
  const int col = pl.lane & 15;
  f4 S = {0, 0, 0, 0};
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    h8 b = h8{0, 0, 0, 0, 0, 0, 0, 0};
    if (col < kTermCols) b = *(const h8 *)(sh.l.terms + col * XR + 32 * i + 8 * pl.kg);
    S = __builtin_amdgcn_mfma_f32_16x16x32_f16(xa[i], b, S, 0, 0, 0);
  }
  const float cnk = sh.l.cn[col & 3];
  const float cm = fmaxf(fmaxf(sh.l.cn[0], sh.l.cn[1]), fmaxf(sh.l.cn[2], sh.l.cn[3]));
  const float cmr = __builtin_amdgcn_sqrtf(cm);
  bool sure = true;
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int t = 16 * pl.wave + 4 * pl.kg + r;
    // columns 0..3 gather their mid and lo terms from columns + 4 and + 8 (row shifts)
    const float tot = fmaf(dppf<0x108>(S[r]), 0x1p-22f, fmaf(dppf<0x104>(S[r]), 0x1p-11f, S[r]));
    const float dk = fmaf(-2.f, tot, cnk);
    const float d0 = dppf<0x00>(dk), d1 = dppf<0x55>(dk), d2 = dppf<0xAA>(dk), d3 = dppf<0xFF>(dk);
    int best = 0;
    float bd = d0, sd = d1;
    if (d1 < bd) { best = 1; bd = d1; sd = d0; }
    if (d2 < bd) { best = 2; sd = bd; bd = d2; } else sd = fminf(sd, d2);
    if (d3 < bd) { best = 3; sd = bd; bd = d3; } else sd = fminf(sd, d3);
    const float xn = sh.l.xn[t];
    const float margin = fmaf(0x1p-13f * xn, cmr, 0x1p-18f * cm);
    if (col < 4) sure = sure & (sd - bd > margin);  // false for NaN
    if (col == 0) sh.l.assign[t] = best;
  }
  if (__syncthreads_or(!sure)) assign_exact(sh);
}

// Deterministic 4-means Lloyd iteration (rows 0, 16, 32, 48 initial, at most 10 rounds),
// then fp16 centroids and ids re-assigned against them.
template <int TENSOR, class S>
__device__ __forceinline__ void encode_centroid(Shared<S::kHalf> &sh, const Place &pl, S &s, uint8_t *dst,
                                                bool cert, double &err, double &nrm) {
  constexpr bool HALF = S::kHalf;
  auto &l = sh.l;
  s.fresh();
  // ---- the block into LDS, the tokens' norms
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int t = 4 * pl.tg + r;
    if constexpr (HALF) {
      *(u4 *)((uint16_t *)l.x + t * XR + 8 * pl.a) = u4{s.w[r][0], s.w[r][1], s.w[r][2], s.w[r][3]};
      float n = 0.f;
#pragma unroll
      for (int e = 0; e < 8; ++e) n = s.square_plus(r, e, n);
      settle(n);
      n = row_sum(n);
      if ((pl.lane & 15) == 0) l.xn[t] = __builtin_amdgcn_sqrtf(n);
    } else {
#pragma unroll
      for (int e = 0; e < 8; ++e) ((double *)l.x)[t * XS + 8 * pl.a + e] = s.v[r][e];
    }
  }
  __syncthreads();
  // ---- wavefront k owns centroid k: channels 2 lane, 2 lane + 1
  double c0 = staged<HALF>(sh, pl.wave * (P / KC), 2 * pl.lane), c1 = staged<HALF>(sh, pl.wave * (P / KC), 2 * pl.lane + 1);
  double *ck = l.c + pl.wave * XS + 2 * pl.lane;
  h8 xa[4];  // MFMA operand of this wavefront's page: token lane & 15, channels 32 i + 8 kg ..
  if constexpr (HALF) {
#pragma unroll
    for (int i = 0; i < 4; ++i)
      xa[i] = *(const h8 *)((const uint16_t *)l.x + (16 * pl.wave + (pl.lane & 15)) * XR + 32 * i + 8 * pl.kg);
  }
  const auto publish = [&]() {  // centroid k as the distances read it
    ck[0] = c0;
    ck[1] = c1;
    if constexpr (HALF) write_terms(sh, pl, c0, c1);
    __syncthreads();
  };
  const auto assign = [&]() {
    if constexpr (HALF) assign_fast(sh, pl, xa);
    else assign_exact(sh);
  };
  publish();
  int prev = -1;
  double a0 = 0.0, a1 = 0.0;  // centroid k's sums
  for (int it = 0; it < 10; ++it) {
    assign();
    const int mine = l.assign[pl.lane];
    const uint64_t moved = __ballot(mine != prev);  // the same in every wavefront
    if (it > 0 && moved == 0) break;  // assignment repeated: converged
    // the sums of fp16 (or decoded) values are exact (see encode_mean), so the tokens that
    // moved update them; tokens with an infinity or NaN go to centroid 0 and stay there
    const uint64_t now = __ballot(mine == pl.wave), was = __ballot(prev == pl.wave);
    prev = mine;
    for (uint64_t m = now & ~was; m; m &= m - 1) {
      const double2 x = staged2<HALF>(sh, __builtin_ctzll(m), pl.lane);
      a0 = a0 + x.x;
      a1 = a1 + x.y;
    }
    for (uint64_t m = was & ~now; m; m &= m - 1) {
      const double2 x = staged2<HALF>(sh, __builtin_ctzll(m), pl.lane);
      a0 = a0 - x.x;
      a1 = a1 - x.y;
    }
    if (now && now != was) {
      const double n = (double)__popcll(now), y = 1.0 / n;
      c0 = div_by(a0, n, y);
      c1 = div_by(a1, n, y);
    }
    __syncthreads();  // every wavefront has read the assignment
    publish();
  }
  // ---- fp16 centroids, and the ids against what is stored
  const uint16_t s0 = canon_zero(f64_to_f16(c0)), s1 = canon_zero(f64_to_f16(c1));
  uint16_t *cc = (uint16_t *)dst;
  if (TENSOR == GKV_KEYS) {
    *(uint32_t *)(cc + pl.wave * D + 2 * pl.lane) = (uint32_t)s0 | ((uint32_t)s1 << 16);
  } else {
    cc[vcent_index(pl.wave, 2 * pl.lane)] = s0;
    cc[vcent_index(pl.wave, 2 * pl.lane + 1)] = s1;
  }
  c0 = f16_to_f64(s0);
  c1 = f16_to_f64(s1);
  __syncthreads();
  publish();
  assign();
  if (threadIdx.x < P / 16) {
    uint32_t w = 0;
    for (int j = 0; j < 16; ++j) w |= (uint32_t)l.assign[threadIdx.x * 16 + j] << (2 * j);
    ((uint32_t *)(dst + KC * D * 2))[threadIdx.x] = w;
  }
  if (cert) {
    int id[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) id[r] = l.assign[4 * pl.tg + r];
    const auto xh = [&](int r, int e) { return l.c[id[r] * XS + 8 * pl.a + e]; };
    float E[4];
    half_errors(s, xh, E);
    block_cert<TENSOR, true>(sh, pl, s, E, half_slack, xh, err, nrm);
  }
}

// Encode the block held in `s` at `level`; with `cert`, err and nrm are the certificate
// numbers of the new record against the source (thread 0; see block_cert).
template <int TENSOR, bool PER_TOKEN, class S>
__device__ __forceinline__ void encode_block(Shared<S::kHalf> &sh, const Place &pl, S &s, uint8_t *dst,
                                             int level, bool cert, double &err, double &nrm) {
  err = nrm = 0.0;
  switch (level) {
    case GKV_EXACT:
      if constexpr (S::kHalf) {
        write_exact<TENSOR>(pl, s, dst);
        const float none[4] = {0.f, 0.f, 0.f, 0.f};
        if (TENSOR != GKV_KEYS && cert)  // no error; the value tensor keeps its row norms
          block_cert<TENSOR, false>(sh, pl, s, none, half_slack, [](int, int) { return 0.0; }, err, nrm);
      }
      break;
    case GKV_INT8:  // never from a decoded record: a demotion lowers the level
      if constexpr (S::kHalf) encode_int<TENSOR, 8, PER_TOKEN>(sh, pl, s, dst, cert, err, nrm);
      break;
    case GKV_INT4: encode_int<TENSOR, 4, PER_TOKEN>(sh, pl, s, dst, cert, err, nrm); break;
    case GKV_INT2: encode_int<TENSOR, 2, PER_TOKEN>(sh, pl, s, dst, cert, err, nrm); break;
    case GKV_CENTROID: encode_centroid<TENSOR>(sh, pl, s, dst, cert, err, nrm); break;
    default: encode_mean<TENSOR>(sh, pl, s, dst, cert, err, nrm); break;
  }
}

}  // namespace enc
}  // namespace gkv
