// Block encoders of the precision ladder (section 3.2), monotone demotion, token
// append, and exact page boxes (section 3.5).
//
// Every arithmetic step whose result is stored (scales, zeros, codes, centroids,
// ids, boxes) is exact-reproducible: fp64 with one rounding per operation, no
// contraction into fused multiply-adds, channel/token-ascending sequential sums,
// and one round-to-nearest-even to fp16 (gkv::f64_to_f16).
#include <hip/hip_runtime.h>

#include "encode_block.h"
#include "gkv_internal.h"

#pragma clang fp contract(off)

using namespace gkv;

namespace {

constexpr int kThreads = enc::kThreads;
using enc::round_up_f32;

// Prefill encode: one workgroup per (block, h, b) of one tensor.  128k tokens x 8 heads of
// the graded ladder: 140 us for the keys, 142 us for the values (352 MB each, 2.5 TB/s;
// 1357 us each with the block staged in LDS and every element's quotient and error in
// fp64).  Vector instructions bound it: 670 a wavefront for int8 and int4 keys, 860 for
// values (row norms as well), 1600-2400 for a centroid block; 32768 tokens x 8 heads take
// 27 us exact, 32-40 us at the int levels, 87-122 us centroid, 24-27 us one-centroid.
// Four wavefronts per SIMD: the keys need 122 registers, the values spill nine words.
template <int TENSOR, bool PER_TOKEN>
__global__ void __launch_bounds__(kThreads, 4) quantize_kernel(const uint16_t *__restrict__ src, int64_t T_src,
                                                            const int8_t *__restrict__ level,
                                                            const int64_t *__restrict__ off, uint8_t *arena,
                                                            int Hkv, int nblk_cap, int blk0, float *cert,
                                                            const int64_t *seq_len) {
  __shared__ enc::Shared<true> sh;
  const int blk = blk0 + blockIdx.x, h = blockIdx.y, b = blockIdx.z;
  const int64_t u = (int64_t)b * Hkv + h;
  // a sequence's own length bounds its rows; blocks past its end are not encoded
  const int64_t Tb = seq_len ? (seq_len[b] < T_src ? seq_len[b] : T_src) : T_src;
  if ((int64_t)blk * P >= Tb) return;
  const int lv = __builtin_amdgcn_readfirstlane((int)level[u * nblk_cap + blk]);
  const enc::Place pl;
  enc::HalfSrc s;
  enc::load_rows(s, pl, src + u * T_src * D, Tb, (int64_t)blk * P);
  double err, nrm;
  enc::encode_block<TENSOR, PER_TOKEN>(sh, pl, s, arena + off[u * nblk_cap + blk], lv, cert != nullptr, err, nrm);
  if (cert && threadIdx.x == 0) {  // error against the exact rows; the value tensor also keeps the row norms
    float *cb = cert + (u * nblk_cap + blk) * 4;
    if (TENSOR == GKV_KEYS) {
      cb[0] = round_up_f32(err);
    } else {
      cb[1] = round_up_f32(err);
      cb[2] = round_up_f32(nrm);
      cb[3] = 0.f;
    }
  }
}

constexpr int kMaxDemoteJobs = 64;
struct DemoteJobs {
  int32_t b[kMaxDemoteJobs], h[kMaxDemoteJobs], blk[kMaxDemoteJobs];
  int8_t to[kMaxDemoteJobs], cur[kMaxDemoteJobs];  // cur from the host mirror: the key
                                                    // workgroup rewrites the device level
  int64_t koff[kMaxDemoteJobs], voff[kMaxDemoteJobs];
};

// Re-encodes the record at `src` (level cur) at `dst` (level to); err as in encode_block.
// The new record may lie over the old one: no wavefront writes before every one has read
// its part (the groups of a token are one wavefront's, so the per-token encoder would
// otherwise write its scales without a barrier).
template <int TENSOR, bool PER_TOKEN>
__device__ __forceinline__ void demote_block(unsigned char *smem, const uint8_t *src, uint8_t *dst, int cur, int to,
                                             bool cert, double &err) {
  const enc::Place pl;
  const auto loaded = [] {  // a barrier alone does not wait for loads in flight
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
  };
  double nrm;
  if (cur == GKV_EXACT) {
    enc::HalfSrc s;
    enc::load_exact<TENSOR>(s, pl, src);
    loaded();
    enc::encode_block<TENSOR, PER_TOKEN>(*reinterpret_cast<enc::Shared<true> *>(smem), pl, s, dst, to, cert, err, nrm);
  } else {
    enc::WideSrc s;
    enc::load_decoded<TENSOR, PER_TOKEN>(s, pl, src, cur);
    loaded();
    enc::encode_block<TENSOR, PER_TOKEN>(*reinterpret_cast<enc::Shared<false> *>(smem), pl, s, dst, to, cert, err,
                                         nrm);
  }
}

// Demotion: grid (jobs, 2 tensors).  Reads the current record through the device
// tables, writes the new record, then points the tables at it.
template <bool PER_TOKEN>
__global__ void __launch_bounds__(kThreads) demote_kernel(DemoteJobs jobs, int8_t *level, int64_t *koff,
                                                          int64_t *voff, uint8_t *arena, int Hkv, int nblk_cap,
                                                          float *cert) {
  extern __shared__ __align__(16) unsigned char smem[];
  const int j = blockIdx.x, tensor = blockIdx.y;
  const int64_t idx = ((int64_t)jobs.b[j] * Hkv + jobs.h[j]) * nblk_cap + jobs.blk[j];
  const int cur = jobs.cur[j], to = jobs.to[j];
  int64_t *offt = tensor == GKV_KEYS ? koff : voff;
  const int64_t dst = tensor == GKV_KEYS ? jobs.koff[j] : jobs.voff[j];
  const uint8_t *src = arena + offt[idx];
  double err;
  if (tensor == GKV_KEYS) demote_block<GKV_KEYS, false>(smem, src, arena + dst, cur, to, cert != nullptr, err);
  else demote_block<GKV_VALUES, PER_TOKEN>(smem, src, arena + dst, cur, to, cert != nullptr, err);
  __syncthreads();  // every thread has read the table entry it is about to change
  if (threadIdx.x == 0) {
    if (cert) {  // the error grows by at most the change of the reconstruction
      float *ce = cert + idx * 4 + (tensor == GKV_KEYS ? 0 : 1);
      *ce = round_up_f32((double)*ce + err);
    }
    offt[idx] = dst;
    if (tensor == GKV_KEYS) level[idx] = jobs.to[j];
  }
}

// Append one token per (b,h); grid (Hkv, B), 128 threads (one per channel).
// The new blocks' slots of the units that open one, and with per-sequence lengths the
// length of every sequence before the token (-1: retired, skipped).
struct NewSlots {
  int64_t k[GKV_MAX_APPEND_UNITS], v[GKV_MAX_APPEND_UNITS];
  int64_t len[GKV_MAX_APPEND_UNITS];
};

// Writes the token of unit u at position T (row tok = T % 64 of the exact block at
// key / value offsets ko / vo, record slot ti): its key and value rows, the value-norm
// bound and, when the token completes a page, that page's box.  128 threads, one per
// channel d.
__device__ __forceinline__ void append_write(const uint16_t *__restrict__ k_new, const uint16_t *__restrict__ v_new,
                                             uint8_t *arena, uint16_t *boxes, int64_t npage_cap, int page,
                                             int64_t u, int64_t T, int64_t ti, int64_t ko, int64_t vo,
                                             bool open_block, float *cert, double *vsq, int d) {
  const int tok = (int)(T % P);
  const uint16_t kv = k_new[u * D + d], vv = v_new[u * D + d];
  if (cert) {  // an exact block: no error; the value norms grow by this row
    const double x = (double)__builtin_bit_cast(_Float16, vv);
    vsq[d] = x * x;
    __syncthreads();
    if (d == 0) {
      double n = 0.0;
      for (int i = 0; i < D; ++i) n += vsq[i];
      float *cb = cert + ti * 4;
      const float vn = round_up_f32(__builtin_sqrt(n));
      if (open_block) {
        cb[0] = 0.f;
        cb[1] = 0.f;
        cb[2] = vn;
        cb[3] = 0.f;
      } else {
        cb[2] = vn > cb[2] ? vn : cb[2];
      }
    }
  }
  // key element (tok, d): page tok>>4, lane ((d>>3)&3)*16 + (tok&15), n = ((d>>5)<<3) | (d&7)
  {
    const int pg = tok >> 4, lane = ((d >> 3) & 3) * 16 + (tok & 15), n = ((d >> 5) << 3) | (d & 7);
    ((uint16_t *)(arena + ko))[(pg * 64 + lane) * 32 + n] = kv;
  }
  // value element (tok, d): page tok>>4, lane ((tok>>2)&3)*16 + (d&15), n = ((d>>4)<<2) | (tok&3)
  {
    const int pg = tok >> 4, lane = ((tok >> 2) & 3) * 16 + (d & 15), n = ((d >> 4) << 2) | (tok & 3);
    ((uint16_t *)(arena + vo))[(pg * 64 + lane) * 32 + n] = vv;
  }
  if (boxes && ((T + 1) % page) == 0) {
    // the page just completed lies in this (exact) block; earlier rows were written
    // by earlier appends, the newest row is still in registers
    const int64_t p = (T + 1) / page - 1;
    const int first = tok + 1 - page;
    _Float16 mn = __builtin_bit_cast(_Float16, kv), mx = mn;
    const uint16_t *rec = (const uint16_t *)(arena + ko);
    for (int t = first; t < tok; ++t) {
      const int pg = t >> 4, lane = ((d >> 3) & 3) * 16 + (t & 15), n = ((d >> 5) << 3) | (d & 7);
      const _Float16 v = __builtin_bit_cast(_Float16, rec[(pg * 64 + lane) * 32 + n]);
      mn = v < mn ? v : mn;
      mx = v > mx ? v : mx;
    }
    uint16_t *bx = boxes + u * npage_cap * 2 * D + box_index(p, d);
    bx[0] = canon_zero(__builtin_bit_cast(uint16_t, mn));
    bx[1] = canon_zero(__builtin_bit_cast(uint16_t, mx));
  }
}

__global__ void __launch_bounds__(128) append_kernel(const uint16_t *__restrict__ k_new,
                                                     const uint16_t *__restrict__ v_new, int8_t *level,
                                                     int64_t *koff, int64_t *voff, uint8_t *arena,
                                                     uint16_t *boxes, int64_t npage_cap, int page, int Hkv,
                                                     int nblk_cap, int64_t T_all, int64_t *seq_len, NewSlots slots,
                                                     float *cert) {
  __shared__ double vsq[D];
  const int h = blockIdx.x, b = blockIdx.y, d = threadIdx.x;
  const int64_t u = (int64_t)b * Hkv + h;
  const int64_t T = seq_len ? slots.len[b] : T_all;
  if (T < 0) return;  // a retired sequence
  if (seq_len && h == 0 && d == 0) seq_len[b] = T + 1;
  const int open_block = (T % P) == 0;
  const int blk = (int)(T / P);
  const int64_t ti = u * nblk_cap + blk;
  int64_t ko, vo;
  if (open_block) {
    ko = slots.k[u];
    vo = slots.v[u];
    if (d == 0) {
      level[ti] = GKV_EXACT;
      koff[ti] = ko;
      voff[ti] = vo;
    }
  } else {
    ko = koff[ti];
    vo = voff[ti];
  }
  if (open_block) {  // a new block's other rows are defined (zero): reads mask them, but 0 * NaN is NaN
    uint4 *kz = (uint4 *)(arena + ko), *vz = (uint4 *)(arena + vo);
    for (int i = d; i < kExactBytes / 16; i += D) {
      kz[i] = make_uint4(0, 0, 0, 0);
      vz[i] = make_uint4(0, 0, 0, 0);
    }
    __syncthreads();
  }
  append_write(k_new, v_new, arena, boxes, npage_cap, page, u, T, ti, ko, vo, open_block, cert, vsq, d);
}

// One decode step's appends for up to kAppendLayers layers of one batch in one launch,
// when no sequence opens a block (the layers share B, Hkv, the block capacity and the
// lengths; the newest block of every unit is exact).  grid (Hkv, B, layers).
constexpr int kAppendLayers = GKV_APPEND_LAYERS;
struct AppendLayer {
  int64_t *koff, *voff;
  uint8_t *arena;
  uint16_t *boxes;
  float *cert;
  int64_t *seq_len;
  int64_t npage_cap;
  int32_t page;
};
struct AppendBatch {
  AppendLayer l[kAppendLayers];
  int64_t len[GKV_MAX_APPEND_UNITS];  // each sequence's length before the step (with per-sequence lengths)
};

__global__ void __launch_bounds__(128) append_layers_kernel(const uint16_t *__restrict__ k_new,
                                                            const uint16_t *__restrict__ v_new, int64_t layer_stride,
                                                            int Hkv, int nblk_cap, int64_t T_all, int ragged,
                                                            AppendBatch ab) {
  __shared__ double vsq[D];
  const int h = blockIdx.x, b = blockIdx.y, l = blockIdx.z, d = threadIdx.x;
  const AppendLayer &L = ab.l[l];
  const int64_t u = (int64_t)b * Hkv + h;
  const int64_t T = ragged ? ab.len[b] : T_all;
  if (T < 0) return;  // a retired sequence
  if (L.seq_len && h == 0 && d == 0) L.seq_len[b] = T + 1;
  const int64_t ti = u * nblk_cap + T / P;
  append_write(k_new + l * layer_stride, v_new + l * layer_stride, L.arena, L.boxes, L.npage_cap, L.page, u, T, ti,
               L.koff[ti], L.voff[ti], false, L.cert, vsq, d);
}

// Page boxes from token-major exact keys; one workgroup per 64 pages of one (b,h).
typedef _Float16 bx8 __attribute__((ext_vector_type(8)));
typedef uint32_t bw4 __attribute__((ext_vector_type(4)));
__global__ void __launch_bounds__(kThreads) boxes_kernel(const uint16_t *__restrict__ k_src, int64_t T_src,
                                                         uint16_t *boxes, int64_t npage_cap, int page, int Hkv,
                                                         int64_t page_begin, int64_t page_end,
                                                         const int64_t *seq_len) {
  __shared__ uint32_t stage[64 * D];  // [channel][page&63] (kmin | kmax << 16)
  const int h = blockIdx.y, b = blockIdx.z;
  const int64_t u = (int64_t)b * Hkv + h;
  const int64_t g0 = (page_begin >> 6) + blockIdx.x;  // box group
  const int64_t p_lo = g0 * 64;
  const uint16_t *src = k_src + u * T_src * D;
  if (seq_len) {  // only the sequence's complete pages
    const int64_t last = seq_len[b] < 0 ? 0 : seq_len[b] / page;
    page_end = page_end < last ? page_end : last;
  }
  // sixteen lanes per page, each with eight channels: sixteen 16-byte streaming row
  // loads in flight per lane, then packed fp16 minima and maxima (exact)
  constexpr int kPagesPerPass = kThreads / 16;
  const int cg = threadIdx.x & 15;
  for (int pi = threadIdx.x >> 4; pi < 64; pi += kPagesPerPass) {
    const int64_t p = p_lo + pi;
    if (p < page_begin || p >= page_end) continue;
    const _Float16 *row = (const _Float16 *)src + p * page * D + 8 * cg;
    bx8 mn, mx;
    for (int t0 = 0; t0 < page; t0 += 16) {
      bx8 v[16];
#pragma unroll
      for (int j = 0; j < 16; ++j) v[j] = __builtin_nontemporal_load((const bx8 *)(row + (int64_t)(t0 + j) * D));
      if (t0 == 0) mn = mx = v[0];
#pragma unroll
      for (int j = 0; j < 16; ++j) {
        mn = __builtin_elementwise_min(mn, v[j]);
        mx = __builtin_elementwise_max(mx, v[j]);
      }
    }
    const bw4 lw = __builtin_bit_cast(bw4, mn), hw = __builtin_bit_cast(bw4, mx);  // channel pairs
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const uint16_t lo = (uint16_t)(lw[e >> 1] >> (16 * (e & 1))), hi = (uint16_t)(hw[e >> 1] >> (16 * (e & 1)));
      stage[(8 * cg + e) * 64 + pi] = (uint32_t)canon_zero(lo) | ((uint32_t)canon_zero(hi) << 16);
    }
  }
  __syncthreads();
  uint32_t *out = (uint32_t *)(boxes + u * npage_cap * 2 * D + box_index(p_lo, 0));
  for (int i = threadIdx.x; i < 64 * D; i += kThreads) {
    const int pi = i & 63;
    const int64_t p = p_lo + pi;
    if (p < page_begin || p >= page_end) continue;
    out[i] = stage[i];
  }
}

// Rate-distortion token scores (section 3.4, Eq. rdscore):
// s_t = a_t * sum_d fl(fl(v_td - v_hat_td)^2), channel-ascending, written as
// order-preserving 64-bit keys.  One wavefront per block, lane = token: the block's
// value record is staged in the wavefront's LDS (an exact record one half of its
// channels at a time) and each lane runs its token's fp64 chain.  v_hat = code *
// scale + zero and v - v_hat are exact in fp64 (all are multiples of 2^-24 below
// 2^26), so forming v_hat with one fused multiply-add gives the same value as a
// product and a sum; the square and each addition round once.  grid (nblk, Hkv, B),
// 64 threads.
//
// Staged words: chunk ck (32 codes, 4 tokens x 8 channels) holds `wpc` words, at most
// four: an int8 record is staged one half of its channels at a time, an exact one a
// quarter.  The 16 chunks of one four-token group c = ck >> 4 are contiguous, and group c
// starts at word c * kRdGroup (4 words of padding after the 16 * 4), so that the lanes of
// the 16 groups, which read the same word of their own group, fall in different banks.
//
// Vector instructions (1135 a wavefront at the graded ladder, conversions at half rate)
// and HBM each take more than half of the time; loads in flight and wavefronts overlap
// them.  The whole selection of 131072 tokens (8 sequences, 4 KV heads, 2% kept) took
// 349.5 us with each lane loading its own 256-byte row, 341.4 us with the rows in 64-byte
// quarters turned in LDS and an int8 record staged whole (11 wavefronts a compute unit),
// 338.3 us as it is (12 wavefronts); with one quarter in flight (15 wavefronts) 353.3 us,
// with the registers held to 128 (15 wavefronts, row loads spilled) 425.8 us.
// A chunk staged in parts shares its lines among them: with plain loads, the next part's
// under way while one is used, the selection of 65536 exact tokens x 16 heads takes 140 us
// (nontemporal, loaded where needed: 209), int8 ones 107 (113).
constexpr int kRdGroup = 16 * 4 + 4;

struct RdShared {
  uint32_t w[16 * kRdGroup];  // staged record words (also the centroids as fp64)
  double2 sz[D];              // per channel: (scale, zero); the one-centroid value in .x
  uint32_t tr[P * 16];        // one quarter of the source rows
};

__device__ __forceinline__ double h2d(uint32_t bits16) {
  return (double)(float)__builtin_bit_cast(_Float16, (uint16_t)bits16);
}

// Stage the 256 chunks of a record, WPC words of each (chunk ck's at word
// ck * src_wpc + src_off of `src`), into the group layout: WPC 16-byte pieces a lane.
// NT: whole chunks, whose lines are read once.
template <bool NT, int WPC>
__device__ __forceinline__ void rd_load(bw4 (&x)[WPC], const uint8_t *src, int src_wpc, int src_off, int lane) {
#pragma unroll
  for (int i = 0; i < WPC; ++i) {
    const int w0 = (i * 64 + lane) * 4;  // staged word index without padding
    const bw4 *at = (const bw4 *)(src + ((int64_t)(w0 / WPC) * src_wpc + src_off + w0 % WPC) * 4);
    x[i] = NT ? __builtin_nontemporal_load(at) : *at;
  }
}
template <int WPC>
__device__ __forceinline__ void rd_store(uint32_t *w, const bw4 (&x)[WPC], int lane) {
  constexpr int gw = 16 * WPC;  // words of one group
#pragma unroll
  for (int i = 0; i < WPC; ++i) {
    const int w0 = (i * 64 + lane) * 4;
    *(bw4 *)(w + (w0 / gw) * kRdGroup + w0 % gw) = x[i];
  }
}

// This lane's code of channel d = 16 j + m (token t: group c = t >> 2, tq = t & 3):
// code n = 4 j + tq of chunk 16 c + m, at bit pos[j & 3] = code_pos(BITS, n) of its word
// (an int8 chunk's words 0..3 or 4..7 are the staged ones).
template <int BITS>
__device__ __forceinline__ uint32_t rd_code(const uint32_t *wl, int j, int m, const int (&pos)[4]) {
  constexpr int wpc = BITS < 4 ? BITS : 4;
  const uint32_t word = wl[m * wpc + 4 * j / (32 / BITS) % wpc];
  return __builtin_amdgcn_ubfe(word, (uint32_t)pos[j & 3], BITS);
}

// The source rows of a block, read in 64-byte row quarters: load r of quarter q takes
// channels 32 q .. of rows 16 r .. 16 r + 15, four lanes a row.  Two quarters are in flight;
// a quarter goes through LDS to the lanes that own its rows.
struct RdRows {
  const uint16_t *at[4];
  bw4 x[2][4];
  __device__ __forceinline__ void load(int q) {
#pragma unroll
    for (int r = 0; r < 4; ++r) x[q & 1][r] = *(const bw4 *)(at[r] + 32 * q);
  }
};

// e += (v_d - v_hat(d))^2 over the channels of quarter q, ascending.  Row t's piece p
// lies at slot p ^ (t >> 2 & 3) of its 64 bytes: the sixteen lanes that a 16-byte access
// serves at once fall on distinct banks, written as well as read.
template <class F>
__device__ __forceinline__ void rd_quarter(double &e, uint32_t *tr, RdRows &rows, int q, int lane, F vhat) {
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int t = 16 * r + (lane >> 2);
    *(bw4 *)(tr + 16 * t + 4 * ((lane & 3) ^ (t >> 2 & 3))) = rows.x[q & 1][r];
  }
  if (q < 2) rows.load(q + 2);
  __syncthreads();
  uint32_t vr[16];
#pragma unroll
  for (int p = 0; p < 4; ++p) {
    const bw4 y = *(const bw4 *)(tr + 16 * lane + 4 * (p ^ (lane >> 2 & 3)));
#pragma unroll
    for (int k = 0; k < 4; ++k) vr[4 * p + k] = y[k];
  }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < 32; ++i) {
    const double v = h2d(vr[i >> 1] >> (16 * (i & 1)));
    const double diff = v - vhat(32 * q + i);
    const double sq = diff * diff;
    e = e + sq;
    // neither LDS reads nor conversions are hoisted past 8 channels (else the unrolled
    // chain keeps those of many more channels in registers)
    if ((i & 7) == 7) {
      asm volatile("" ::: "memory");
      __builtin_amdgcn_sched_barrier(0);
    }
  }
}

template <class F>
__device__ __forceinline__ void rd_chain(double &e, uint32_t *tr, RdRows &rows, int lane, F vhat) {
#pragma unroll
  for (int q = 0; q < 4; ++q) rd_quarter(e, tr, rows, q, lane, vhat);
}

// The chain over a record staged in 4 / Q parts of Q row quarters, the next part in flight.
template <int Q, class F>
__device__ __forceinline__ void rd_chain_parts(double &e, RdShared &S, RdRows &rows, const uint8_t *src,
                                               int src_wpc, int lane, F vhat) {
  bw4 x[4];
  rd_load<false>(x, src, src_wpc, 0, lane);
#pragma unroll
  for (int q0 = 0; q0 < 4; q0 += Q) {
    rd_store(S.w, x, lane);
    if (q0 + Q < 4) rd_load<false>(x, src, src_wpc, 4 * (q0 / Q + 1), lane);
    __syncthreads();
#pragma unroll
    for (int q = q0; q < q0 + Q; ++q) rd_quarter(e, S.tr, rows, q, lane, vhat);
    __syncthreads();
  }
}

__global__ void __launch_bounds__(64) rd_score_kernel(const uint16_t *__restrict__ v_src,
                                                      const float *__restrict__ mass, int64_t T,
                                                      const int8_t *__restrict__ level,
                                                      const int64_t *__restrict__ voff,
                                                      const uint8_t *__restrict__ arena, int Hkv, int nblk_cap,
                                                      uint64_t *__restrict__ keys, int64_t key_stride, int vtok) {
  __shared__ __align__(16) RdShared S;
  const int blk = blockIdx.x, h = blockIdx.y, b = blockIdx.z;
  const int lane = threadIdx.x, c = lane >> 2, tq = lane & 3;
  const int64_t u = (int64_t)b * Hkv + h;
  const int64_t ti = u * nblk_cap + blk;
  const int64_t tok = (int64_t)blk * P + lane;
  const int lv = level[ti];
  const uint8_t *rec = arena + voff[ti];

  RdRows rows;
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int64_t t = (int64_t)blk * P + 16 * r + (lane >> 2);  // rows past T: the last row, not stored
    rows.at[r] = v_src + (u * T + (t < T ? t : T - 1)) * D + 8 * (lane & 3);
  }
  rows.load(0);
  rows.load(1);
  const double a = (double)mass[u * T + (tok < T ? tok : T - 1)];

  double e = 0.0;
  const uint32_t *wl = S.w + c * kRdGroup;
  if (lv == GKV_EXACT) {  // chunk ck: 64 B; channels 16 j + m of token 4 c + tq at half 4 j + tq of chunk 16 c + m
    const uint32_t *wh = wl + (tq >> 1);
    const int sh = 16 * (tq & 1);
    rd_chain_parts<1>(e, S, rows, rec, 16, lane, [&](int d) { return h2d(wh[(d & 15) * 4 + 2 * (d >> 4 & 1)] >> sh); });
  } else if (lv == GKV_MEAN || lv == GKV_CENTROID) {
    const uint16_t *cc = (const uint16_t *)rec;
    if (lv == GKV_MEAN) {
      for (int d = lane; d < D; d += 64) S.sz[d].x = h2d(cc[d]);
      __syncthreads();
      rd_chain(e, S.tr, rows, lane, [&](int d) { return S.sz[d].x; });
    } else {
      double *cent = (double *)S.w;  // [KC][D + 1]
      for (int i = lane; i < KC * D; i += 64) {
        const int k = i >> 7, d = i & 127;
        cent[k * (D + 1) + d] = h2d(cc[vcent_index(k, d)]);
      }
      const int id = (rec[KC * D * 2 + (lane >> 2)] >> (2 * (lane & 3))) & 3;
      __syncthreads();
      const double *ct = cent + id * (D + 1);
      rd_chain(e, S.tr, rows, lane, [&](int d) { return ct[d]; });
    }
  } else {  // int8 / int4 / int2: (scale, zero) per channel or per token, then the codes
    const uint16_t *sz = (const uint16_t *)rec;
    double s = 0.0, z = 0.0;
    if (vtok) {
      s = h2d(sz[lane]);
      z = h2d(sz[P + lane]);
    } else {
      for (int e2 = lane; e2 < D; e2 += 64) S.sz[sz_channel(GKV_VALUES, e2)] = make_double2(h2d(sz[e2]), h2d(sz[D + e2]));
    }
    int pos[4];  // bit positions of this lane's codes (the same every four channel groups j)
#pragma unroll
    for (int r = 0; r < 4; ++r) pos[r] = code_pos(lv, 4 * r + tq);
    const uint8_t *codes = rec + kSZBytes;
#define GKV_RD_INT(BITS, CHAIN, ...)                                                                        \
  if (vtok)                                                                                                 \
    CHAIN(e, __VA_ARGS__, [&](int d) { return __builtin_fma((double)rd_code<BITS>(wl, d >> 4, d & 15, pos), s, z); }); \
  else                                                                                                      \
    CHAIN(e, __VA_ARGS__, [&](int d) {                                                                      \
      const double2 g = S.sz[d];                                                                            \
      return __builtin_fma((double)rd_code<BITS>(wl, d >> 4, d & 15, pos), g.x, g.y);                       \
    })
    if (lv == GKV_INT8) {
      GKV_RD_INT(8, rd_chain_parts<2>, S, rows, codes, 8, lane);
    } else if (lv == GKV_INT4) {
      bw4 x[4];
      rd_load<true>(x, codes, 4, 0, lane);
      rd_store(S.w, x, lane);
      __syncthreads();
      GKV_RD_INT(4, rd_chain, S.tr, rows, lane);
    } else {
      bw4 x[2];
      rd_load<true>(x, codes, 2, 0, lane);
      rd_store(S.w, x, lane);
      __syncthreads();
      GKV_RD_INT(2, rd_chain, S.tr, rows, lane);
    }
#undef GKV_RD_INT
  }
  if (tok < T) {
    double sc = a * e;
    sc = sc + 0.0;  // -0 -> +0
    uint64_t bits;
    __builtin_memcpy(&bits, &sc, 8);
    keys[u * key_stride + tok] = (bits >> 63) ? ~bits : (bits | 0x8000000000000000ull);
  }
}

}  // namespace

void gkv_launch_rd_score(const gkv_cache *c, const uint16_t *v_src, const float *mass, uint64_t *keys,
                         int64_t key_stride, hipStream_t stream) {
  const int nblk = (int)((c->T + P - 1) / P);
  hipLaunchKernelGGL(rd_score_kernel, dim3(nblk, c->Hkv, c->B), dim3(64), 0, stream, v_src,
                     mass, c->T, c->level, c->voff, c->arena, c->Hkv, c->nblk_cap, keys, key_stride, c->v_per_token);
}

// ---------------------------------------------------------------- C ABI
static gkv_status hip_status() { return hipGetLastError() == hipSuccess ? GKV_OK : GKV_E_HIP; }

__global__ void set_len_kernel(int64_t *seq_len, int b, int64_t v) {
  if (threadIdx.x == 0) seq_len[b] = v;
}

gkv_status gkv_launch_set_len(int64_t *seq_len, int b, int64_t v, hipStream_t stream) {
  hipLaunchKernelGGL(set_len_kernel, dim3(1), dim3(64), 0, stream, seq_len, b, v);
  return hip_status();
}

extern "C" gkv_status gkv_quantize_block(const gkv_cache *c, int32_t which, const uint16_t *src, int64_t T_src,
                                         int32_t blk_begin, int32_t blk_end, void *stream) {
  gkv_status st = gkv_validate_cache(c);
  if (st) return st;
  if (!src || (which != GKV_KEYS && which != GKV_VALUES) || T_src <= 0) return GKV_E_ARG;
  if (blk_begin < 0 || blk_end > c->nblk_cap || blk_begin > blk_end) return GKV_E_SHAPE;
  if (blk_begin == blk_end) return GKV_OK;
  for (int b = 0; b < c->B; ++b) {
    // with per-sequence lengths the sequence's own length bounds its blocks
    const int64_t Tb = c->seq_len_host ? c->seq_len_host[b] : T_src;
    if (Tb > T_src) return GKV_E_SHAPE;
    for (int h = 0; h < c->Hkv; ++h)
      for (int blk = blk_begin; blk < blk_end; ++blk) {
        if (c->seq_len_host && (int64_t)blk * P >= Tb) continue;  // not encoded
        const int lv = c->level_host[((int64_t)b * c->Hkv + h) * c->nblk_cap + blk];
        if (level_rank(lv) < 0) return GKV_E_ARG;
        if ((int64_t)(blk + 1) * P > Tb && lv != GKV_EXACT) return GKV_E_SHAPE;
        if ((int64_t)blk * P >= Tb) return GKV_E_SHAPE;
      }
  }
  dim3 grid(blk_end - blk_begin, c->Hkv, c->B);
#define GKV_QUANT(t, vt)                                                                                            \
  hipLaunchKernelGGL((quantize_kernel<t, vt>), grid, dim3(kThreads), 0, (hipStream_t)stream, src, T_src, c->level,  \
                     t == GKV_KEYS ? c->koff : c->voff, c->arena, c->Hkv, c->nblk_cap, blk_begin, c->cert,          \
                     (const int64_t *)c->seq_len)
  if (which == GKV_KEYS) GKV_QUANT(GKV_KEYS, false);
  else if (c->v_per_token) GKV_QUANT(GKV_VALUES, true);
  else GKV_QUANT(GKV_VALUES, false);
#undef GKV_QUANT
  return hip_status();
}

extern "C" gkv_status gkv_demote(gkv_cache *c, int32_t n, const int32_t *jobs, const int8_t *to,
                                 const int64_t *nk, const int64_t *nv, void *stream) {
  gkv_status st = gkv_validate_cache(c);
  if (st) return st;
  if (n < 0) return GKV_E_ARG;
  if (n == 0) return GKV_OK;
  if (!jobs || !to || !nk || !nv) return GKV_E_ARG;
  const int64_t nblk = (c->T + P - 1) / P;
  for (int i = 0; i < n; ++i) {
    const int b = jobs[3 * i], h = jobs[3 * i + 1], blk = jobs[3 * i + 2];
    if (b < 0 || b >= c->B || h < 0 || h >= c->Hkv || blk < 0 || blk >= nblk) return GKV_E_SHAPE;
    const int cur = c->level_host[((int64_t)b * c->Hkv + h) * c->nblk_cap + blk];
    if (level_rank(to[i]) < 0) return GKV_E_ARG;
    if (level_rank(to[i]) >= level_rank(cur)) return GKV_E_NOT_MONOTONE;
    if ((int64_t)(blk + 1) * P > seq_tokens(c, b)) return GKV_E_SHAPE;  // a partial block stays exact
    const int64_t bb = block_bytes(to[i]);
    if (nk[i] < 0 || nv[i] < 0 || nk[i] + bb > c->arena_bytes || nv[i] + bb > c->arena_bytes) return GKV_E_ARG;
    for (int j = 0; j < i; ++j)
      if (jobs[3 * j] == b && jobs[3 * j + 1] == h && jobs[3 * j + 2] == blk) return GKV_E_ARG;
  }
  for (int base = 0; base < n; base += kMaxDemoteJobs) {
    const int cnt = n - base < kMaxDemoteJobs ? n - base : kMaxDemoteJobs;
    DemoteJobs J;
    for (int i = 0; i < cnt; ++i) {
      J.b[i] = jobs[3 * (base + i)];
      J.h[i] = jobs[3 * (base + i) + 1];
      J.blk[i] = jobs[3 * (base + i) + 2];
      J.to[i] = to[base + i];
      J.cur[i] = c->level_host[((int64_t)J.b[i] * c->Hkv + J.h[i]) * c->nblk_cap + J.blk[i]];
      J.koff[i] = nk[base + i];
      J.voff[i] = nv[base + i];
    }
    constexpr size_t lds = sizeof(enc::Shared<false>) > sizeof(enc::Shared<true>) ? sizeof(enc::Shared<false>)
                                                                                   : sizeof(enc::Shared<true>);
    if (c->v_per_token)
      hipLaunchKernelGGL(demote_kernel<true>, dim3(cnt, 2), dim3(kThreads), lds, (hipStream_t)stream, J, c->level,
                         c->koff, c->voff, c->arena, c->Hkv, c->nblk_cap, c->cert);
    else
      hipLaunchKernelGGL(demote_kernel<false>, dim3(cnt, 2), dim3(kThreads), lds, (hipStream_t)stream, J, c->level,
                         c->koff, c->voff, c->arena, c->Hkv, c->nblk_cap, c->cert);
    if (hipGetLastError() != hipSuccess) return GKV_E_HIP;
  }
  for (int i = 0; i < n; ++i)
    c->level_host[((int64_t)jobs[3 * i] * c->Hkv + jobs[3 * i + 1]) * c->nblk_cap + jobs[3 * i + 2]] = to[i];
  gkv_stamp(c);
  return GKV_OK;
}

extern "C" gkv_status gkv_page_boxes(const gkv_cache *c, const uint16_t *k_src, int64_t T_src,
                                     int64_t page_begin, int64_t page_end, void *stream) {
  gkv_status st = gkv_validate_cache(c);
  if (st) return st;
  if (!c->page || !k_src) return GKV_E_ARG;
  if (page_begin < 0 || page_begin > page_end || page_end > c->npage_cap) return GKV_E_SHAPE;
  if (page_end * c->page > T_src) return GKV_E_SHAPE;
  if (page_begin == page_end) return GKV_OK;
  const int64_t g0 = page_begin >> 6, g1 = (page_end + 63) >> 6;
  dim3 grid((unsigned)(g1 - g0), c->Hkv, c->B);
  hipLaunchKernelGGL(boxes_kernel, grid, dim3(kThreads), 0, (hipStream_t)stream, k_src, T_src, c->boxes,
                     c->npage_cap, c->page, c->Hkv, page_begin, page_end, (const int64_t *)c->seq_len);
  return hip_status();
}

extern "C" gkv_status gkv_append(gkv_cache *c, const uint16_t *k_new, const uint16_t *v_new,
                                 const int64_t *new_koff, const int64_t *new_voff, void *stream) {
  gkv_status st = gkv_validate_cache(c);
  if (st) return st;
  if (!k_new || !v_new) return GKV_E_ARG;
  const int64_t units = (int64_t)c->B * c->Hkv;
  if (c->seq_len_host && c->B > GKV_MAX_APPEND_UNITS) return GKV_E_UNSUPPORTED;
  NewSlots slots;
  bool any_open = false;
  for (int b = 0; b < c->B; ++b) {
    const int64_t T = seq_tokens(c, b);
    if (c->seq_len_host) slots.len[b] = T;
    if (T < 0) continue;  // retired
    const int blk = (int)(T / P);
    if (blk >= c->nblk_cap) return GKV_E_SHAPE;
    if (c->page && (T + 1) / c->page > c->npage_cap) return GKV_E_SHAPE;
    const bool open = (T % P) == 0;
    any_open |= open;
    for (int h = 0; h < c->Hkv; ++h) {
      const int64_t u = (int64_t)b * c->Hkv + h;
      if (open) {
        if (units > GKV_MAX_APPEND_UNITS) return GKV_E_UNSUPPORTED;
        if (!new_koff || !new_voff) return GKV_E_ARG;
        if (new_koff[u] < 0 || new_voff[u] < 0 || new_koff[u] + kExactBytes > c->arena_bytes ||
            new_voff[u] + kExactBytes > c->arena_bytes)
          return GKV_E_ARG;
        slots.k[u] = new_koff[u];
        slots.v[u] = new_voff[u];
      } else if (c->level_host[u * c->nblk_cap + blk] != GKV_EXACT) {
        return GKV_E_ARG;
      }
    }
  }
  hipLaunchKernelGGL(append_kernel, dim3(c->Hkv, c->B), dim3(128), 0, (hipStream_t)stream, k_new, v_new, c->level,
                     c->koff, c->voff, c->arena, c->page ? c->boxes : nullptr, c->npage_cap, c->page ? c->page : 1,
                     c->Hkv, c->nblk_cap, c->T, c->seq_len, slots, c->cert);
  if (hipGetLastError() != hipSuccess) return GKV_E_HIP;
  gkv_append_commit(c, any_open);
  return GKV_OK;
}

// The host side of an enqueued append: the opened blocks' levels, the lengths and T.
void gkv_append_commit(gkv_cache *c, bool any_open) {
  int64_t mx = 0;
  for (int b = 0; b < c->B; ++b) {
    const int64_t T = seq_tokens(c, b);
    if (T < 0) continue;
    if (T % P == 0)
      for (int h = 0; h < c->Hkv; ++h) c->level_host[((int64_t)b * c->Hkv + h) * c->nblk_cap + T / P] = GKV_EXACT;
    if (c->seq_len_host) c->seq_len_host[b] = T + 1;
    mx = T + 1 > mx ? T + 1 : mx;
  }
  c->T = c->seq_len_host ? mx : c->T + 1;
  // the tables change only when a block opens; a dense plan covers whole blocks, and
  // the attention masks a block's tokens past the length at run time
  if (any_open) gkv_stamp(c);
}

// One launch for n <= GKV_APPEND_LAYERS layers of a step that opens no block (k_new,
// v_new: their rows, layer after layer): the caller has checked what gkv_append
// checks (same B, Hkv, capacity and lengths over the layers; every newest block
// exact; page-box capacity).  Nothing of the host state changes.
gkv_status gkv_launch_append_layers(gkv_cache *const *caches, int n, const uint16_t *k_new, const uint16_t *v_new,
                                    hipStream_t stream) {
  const gkv_cache *c0 = caches[0];
  if (n < 1 || n > kAppendLayers) return GKV_E_ARG;
  if (c0->seq_len_host && c0->B > GKV_MAX_APPEND_UNITS) return GKV_E_UNSUPPORTED;
  const int64_t stride = (int64_t)c0->B * c0->Hkv * D;
  AppendBatch ab;
  for (int i = 0; i < n; ++i) {
    const gkv_cache *c = caches[i];
    ab.l[i] = AppendLayer{c->koff, c->voff, c->arena, c->page ? c->boxes : nullptr, c->cert, c->seq_len,
                          c->npage_cap, c->page ? c->page : 1};
  }
  if (c0->seq_len_host)
    for (int b = 0; b < c0->B; ++b) ab.len[b] = c0->seq_len_host[b];
  hipLaunchKernelGGL(append_layers_kernel, dim3(c0->Hkv, c0->B, n), dim3(128), 0, stream, k_new, v_new, stride,
                     c0->Hkv, c0->nblk_cap, c0->T, c0->seq_len_host ? 1 : 0, ab);
  return hipGetLastError() == hipSuccess ? GKV_OK : GKV_E_HIP;
}
