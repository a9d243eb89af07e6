// Lossless acceptance kernels (Sec. 3): greedy arg-max / longest matching prefix / bonus
// token, and the speculative-sampling variant with supplied uniforms.
//
// Both are one streaming pass over [rows][vocab] logits, so the vocabulary of every row
// is cut into segments and one work-group reduces one (row, segment); a small epilogue
// per sequence merges the segment results and walks the verify rows.
#include "fd_common.h"
#include <float.h>
#include <type_traits>

namespace fd {

constexpr int ACC_BLOCK = 256;

// Reductions by the register file's own lane shifts (DPP).  Every kernel here ends in a chain of them that nothing overlaps, and a
// step through LDS (__shfl_xor) is a latency of LDS.  us a call, through LDS -> by lane shifts, bf16 rows of 151936: greedy acceptance
// of 8 rows 6.45 -> 5.95, of 128 11.1 -> 10.8; sampling of 4 pairs of rows 14.8 -> 13.7; selection over 8 rows 9.0 -> 8.4.
// wave_*: over the wave, the result in every lane (all lanes active).  row_*: over each row of sixteen lanes, the result in all of them.
template <int CTRL, int ROWS = 0xf> __device__ __forceinline__ int lane_shift(int old, int v) {
  return __builtin_amdgcn_update_dpp(old, v, CTRL, ROWS, 0xf, false);
}
template <int CTRL, int ROWS = 0xf> __device__ __forceinline__ float lane_shift(float old, float v) {
  return __int_as_float(lane_shift<CTRL, ROWS>(__float_as_int(old), __float_as_int(v)));
}
template <int CTRL, int ROWS = 0xf> __device__ __forceinline__ double lane_shift(double old, double v) {
  return __hiloint2double(lane_shift<CTRL, ROWS>(__double2hiint(old), __double2hiint(v)), lane_shift<CTRL, ROWS>(__double2loint(old), __double2loint(v)));
}
__device__ __forceinline__ int last_lane(int v) { return __builtin_amdgcn_readlane(v, 63); }
__device__ __forceinline__ float last_lane(float v) { return __int_as_float(last_lane(__float_as_int(v))); }
__device__ __forceinline__ double last_lane(double v) { return __hiloint2double(last_lane(__double2hiint(v)), last_lane(__double2loint(v))); }
// lane i: op over lanes 0 .. i (shifts by 1, 2, 4, 8 within the rows, then the last lane of a row to the next one, of the lower half to the
// upper); `none`: a value that op leaves the other as it is with
template <typename T, typename Op> __device__ __forceinline__ T wave_scan(T v, T none, Op op) {
  v = op(v, lane_shift<0x111>(none, v));
  v = op(v, lane_shift<0x112>(none, v));
  v = op(v, lane_shift<0x114>(none, v));
  v = op(v, lane_shift<0x118>(none, v));
  v = op(v, lane_shift<0x142, 0xa>(none, v));
  return op(v, lane_shift<0x143, 0xc>(none, v));
}
template <typename T, typename Op> __device__ __forceinline__ T row_all(T v, Op op) {        // rotations by 8, 4, 2, 1
  v = op(v, lane_shift<0x128>(v, v));
  v = op(v, lane_shift<0x124>(v, v));
  v = op(v, lane_shift<0x122>(v, v));
  return op(v, lane_shift<0x121>(v, v));
}
__device__ __forceinline__ float wave_max(float v) { return last_lane(wave_scan(v, -INFINITY, [](float a, float b) { return fmaxf(a, b); })); }
__device__ __forceinline__ int wave_min(int v) { return last_lane(wave_scan(v, 0x7fffffff, [](int a, int b) { return min(a, b); })); }
__device__ __forceinline__ double wave_prefix(double v) { return wave_scan(v, 0.0, [](double a, double b) { return a + b; }); }
__device__ __forceinline__ double wave_sum(double v) { return last_lane(wave_prefix(v)); }
__device__ __forceinline__ float row_max(float v) { return row_all(v, [](float a, float b) { return fmaxf(a, b); }); }
__device__ __forceinline__ double row_max(double v) { return row_all(v, [](double a, double b) { return fmax(a, b); }); }
__device__ __forceinline__ int row_min(int v) { return row_all(v, [](int a, int b) { return min(a, b); }); }
__device__ __forceinline__ double row_sum(double v) { return row_all(v, [](double a, double b) { return a + b; }); }

// Eight consecutive logits of a row as they lie in memory.  Requesting and widening are separate steps: a kernel requests every
// vector of its share first and widens them afterwards, so that all of its bytes are in flight together.  (Widened where it
// was loaded, behind a test of alignment or bounds, each vector waited for the one before it.  us, before -> after, over rows
// of 151936 bf16 logits: arg-max of 128 rows 11.0 -> 9.3, draft statistics of 480 29.7 -> 23.9 (6.1 TB/s), sampling statistics of
// 64 pairs of rows 14.1 -> 10.9.)  Requests are unconditional: 16-byte loads at any alignment, moved down to end at the
// share's end.
template <typename T> struct Vec8;
template <> struct Vec8<bf16_t> { u32x4 w; };
template <> struct Vec8<float> { f32x4 a, b; };

__device__ __forceinline__ void fetch8(const bf16_t* p, Vec8<bf16_t>& r) {
  typedef u32x4 __attribute__((aligned(2))) u32x4_any;
  r.w = __builtin_nontemporal_load(reinterpret_cast<const u32x4_any*>(p));
}
__device__ __forceinline__ void fetch8(const float* p, Vec8<float>& r) {
  typedef f32x4 __attribute__((aligned(4))) f32x4_any;
  r.a = __builtin_nontemporal_load(reinterpret_cast<const f32x4_any*>(p));
  __builtin_amdgcn_sched_barrier(0);
  r.b = __builtin_nontemporal_load(reinterpret_cast<const f32x4_any*>(p) + 1);
}
// near the end of a row, or in a row of fewer than eight logits: one by one, the last one repeated
__device__ __forceinline__ void fetch8_short(const bf16_t* row, int e, int end, Vec8<bf16_t>& r) {
#pragma unroll
  for (int i = 0; i < 4; ++i) r.w[i] = (unsigned)row[min(e + 2 * i, end - 1)] | (unsigned)row[min(e + 2 * i + 1, end - 1)] << 16;
}
__device__ __forceinline__ void fetch8_short(const float* row, int e, int end, Vec8<float>& r) {
#pragma unroll
  for (int i = 0; i < 4; ++i) { r.a[i] = row[min(e + i, end - 1)]; r.b[i] = row[min(e + 4 + i, end - 1)]; }
}
__device__ __forceinline__ void widen8(const Vec8<bf16_t>& r, float (&x)[8]) {
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    x[2 * i] = __uint_as_float(r.w[i] << 16);
    x[2 * i + 1] = __uint_as_float(r.w[i] & 0xffff0000u);
  }
}
__device__ __forceinline__ void widen8(const Vec8<float>& r, float (&x)[8]) {
#pragma unroll
  for (int i = 0; i < 4; ++i) { x[i] = r.a[i]; x[4 + i] = r.b[i]; }
}

__device__ __forceinline__ void hold8(Vec8<bf16_t>& r) { asm volatile("" : "+v"(r.w)); }
__device__ __forceinline__ void hold8(Vec8<float>& r) { asm volatile("" : "+v"(r.a), "+v"(r.b)); }

// A thread's share of [e0, end) of a row: N vectors, the u-th from element at(u) on.  A vector that would leave the share is
// moved down to end there (in the row's last share also where that begins before it): it then repeats elements of the
// row, which a maximum and its lowest index do not mind; a sum counts the vector's own elements only.
// SHORT: rows of fewer than eight logits.
template <typename T, int N, bool SHORT> struct RowShare {
  int e0, end;
  Vec8<T> r[N];
  __device__ __forceinline__ RowShare(int e0_, int end_) : e0(e0_), end(end_) {}
  __device__ __forceinline__ int at(int u) const { return e0 + (u * ACC_BLOCK + (int)threadIdx.x) * 8; }
  __device__ __forceinline__ int from(int u) const { return SHORT ? at(u) : min(at(u), end - 8); }      // first element held
  __device__ __forceinline__ void request(const T* row) {
#pragma unroll
    for (int u = 0; u < N; ++u) {
      if (SHORT) fetch8_short(row, at(u), end, r[u]); else fetch8(row + from(u), r[u]);
    }
    // (without the two barriers the halves of a vector of floats go out in reverse, the last one when all the others have landed:
    // selection over 40 rows of 151936 floats 13.5 us a call, now 12.6)
    if (sizeof(T) == 4) __builtin_amdgcn_sched_barrier(0);
  }
  // Before a second pass over the vectors: keeps the compiler from holding the first pass's widened floats (twice the registers).
  __device__ __forceinline__ void again() {
#pragma unroll
    for (int u = 0; u < N; ++u) if (sizeof(T) == 2) hold8(r[u]);
  }
  __device__ __forceinline__ float max() const {
    float m = -INFINITY;
#pragma unroll
    for (int u = 0; u < N; ++u) {
      float x[8];
      widen8(r[u], x);
#pragma unroll
      for (int i = 0; i < 8; ++i) m = fmaxf(m, x[i]);
    }
    return m;
  }
  __device__ __forceinline__ int lowest_index_of(float v) const {      // 0x7fffffff: not held
    int bi = 0x7fffffff;
#pragma unroll
    for (int u = N - 1; u >= 0; --u) {
      float x[8];
      widen8(r[u], x);
#pragma unroll
      for (int i = 7; i >= 0; --i) if (x[i] == v) bi = from(u) + i;    // descending walk: the lowest index is kept
    }
    return bi;
  }
  template <typename F> __device__ __forceinline__ float sum(F&& f) const {
    float tot = 0.f;
#pragma unroll
    for (int u = 0; u < N; ++u) {
      float x[8], t = 0.f;
      widen8(r[u], x);
      if (!SHORT && sizeof(T) == 4) {              // (floats: a test per element costs less than a branch per vector, bf16 the other way round)
        const int skip = at(u) - from(u);
#pragma unroll
        for (int i = 0; i < 8; ++i) t += i >= skip ? f(x[i]) : 0.f;
        tot += t;
        continue;
      }
#pragma unroll
      for (int i = 0; i < 8; ++i) t += f(x[i]);
      if (at(u) + 8 > end) {                       // few lanes of a share's last vector, and all beyond
        t = 0.f;
        for (int i = 0; i < 8; ++i) {
          const int e = from(u) + i;
          if (e >= at(u) && e < end) t += f(x[i]);
        }
      }
      tot += t;
    }
    return tot;
  }
};

// Elements e .. e + 7 (e < vocab) of two rows as floats, -inf past the end; both are in flight together.
template <typename T>
__device__ __forceinline__ void load_pair8(const T* a, const T* b, int e, int vocab, float (&xa)[8], float (&xb)[8]) {
  Vec8<T> ra, rb;
  if (e + 8 <= vocab) { fetch8(a + e, ra); fetch8(b + e, rb); }
  else { fetch8_short(a, e, vocab, ra); fetch8_short(b, e, vocab, rb); }
  widen8(ra, xa); widen8(rb, xb);
  if (e + 8 > vocab) {
#pragma unroll
    for (int i = 0; i < 8; ++i) if (e + i >= vocab) { xa[i] = -INFINITY; xb[i] = -INFINITY; }
  }
}

// (value, index) with "larger value wins, equal values: lower index wins"
__device__ __forceinline__ void amax_merge(float& v, int& i, float ov, int oi) {
  if (ov > v || (ov == v && oi < i)) { v = ov; i = oi; }
}

// ---------------------------------------------------------------------------------------
// Greedy, pass 1: arg-max of one vocabulary segment of one row.
//   grid (segments, rows); part_val/part_idx [rows][segments]
// A segment is at most ACC_BLOCK * 8 * NR logits (NR <= ARG_ROUNDS rounds), so a lane holds all of its share in
// registers.  First the segment's maximum (one max per logit), then only the lanes whose own
// maximum equals it look for the lowest index holding that value: comparing (value, index)
// pairs logit by logit would cost several times the instructions and bound the kernel by
// arithmetic rather than by the stream.
// ---------------------------------------------------------------------------------------
constexpr int ARG_ROUNDS = 5;

template <typename T, int NR, bool SHORT>
__global__ __launch_bounds__(ACC_BLOCK) void argmax_partial_kernel(
    const T* __restrict__ logits, long long row_stride, int vocab, int seg_len,
    float* __restrict__ part_val, int* __restrict__ part_idx) {
  const int seg = blockIdx.x, row = blockIdx.y, nseg = gridDim.x;
  const T* rp = logits + (long long)row * row_stride;
  const int e0 = seg * seg_len;
  RowShare<T, NR, SHORT> sh(e0, min(vocab, e0 + min(seg_len, NR * ACC_BLOCK * 8)));
  __shared__ float sv[ACC_BLOCK / FD_WAVE]; __shared__ int si[ACC_BLOCK / FD_WAVE];
  sh.request(rp);
  const float m = sh.max();
  const float wm = wave_max(m);
  if ((threadIdx.x & 63) == 0) sv[threadIdx.x >> 6] = wm;
  __syncthreads();
  float M = sv[0];
#pragma unroll
  for (int w = 1; w < ACC_BLOCK / FD_WAVE; ++w) M = fmaxf(M, sv[w]);
  int bi = 0x7fffffff;
  sh.again();
  if (m == M) bi = sh.lowest_index_of(M);
  bi = wave_min(bi);
  if ((threadIdx.x & 63) == 0) si[threadIdx.x >> 6] = bi;
  __syncthreads();
  if (threadIdx.x == 0) {
#pragma unroll
    for (int w = 1; w < ACC_BLOCK / FD_WAVE; ++w) bi = min(bi, si[w]);
    part_val[(long long)row * nseg + seg] = M;
    part_idx[(long long)row * nseg + seg] = bi;
  }
}

// ---------------------------------------------------------------------------------------
// Greedy, pass 2: one wave per sequence.  Merge the segment results of each verify row,
// then count the leading rows whose arg-max equals the token fed at the next row.
// ---------------------------------------------------------------------------------------
constexpr int GE_GROUP = 16;                       // lanes that merge one row's segments
constexpr int GE_ROWS = ACC_BLOCK / GE_GROUP;     // rows merged at a time

__global__ __launch_bounds__(ACC_BLOCK) void accept_greedy_epilogue_kernel(
    const float* __restrict__ part_val, const int* __restrict__ part_idx, int nseg,
    const int* __restrict__ row_indptr, const int* __restrict__ input_tokens,
    int total_rows, int max_rows_per_seq,
    int* __restrict__ accept_len, int* __restrict__ bonus_token, int* __restrict__ row_argmax) {
  const int seq = blockIdx.x, grp = threadIdx.x / GE_GROUP, gl = threadIdx.x % GE_GROUP;
  int r0 = clampi(row_indptr[seq], 0, total_rows);
  int k = clampi(row_indptr[seq + 1] - r0, 0, min(max_rows_per_seq, total_rows - r0));
  if (k == 0) { if (threadIdx.x == 0) { accept_len[seq] = 0; bonus_token[seq] = -1; } return; }
  // Rows GE_ROWS at a time, in order: GE_GROUP lanes merge a row's segments (every load of a batch is
  // in flight together); the first row whose arg-max differs from the token fed at the next row --
  // or the last row -- ends the step and its arg-max is the bonus token.
  __shared__ int s_first_bad, s_bonus;
  if (threadIdx.x == 0) { s_first_bad = 0x7fffffff; s_bonus = -1; }
  __syncthreads();
  bool done = false;
  for (int j0 = 0; j0 < k; j0 += GE_ROWS) {
    const int j = j0 + grp;
    float bv = -INFINITY; int bi = 0x7fffffff;
    if (j < k)
      for (int s = gl; s < nseg; s += GE_GROUP)
        amax_merge(bv, bi, part_val[(long long)(r0 + j) * nseg + s], part_idx[(long long)(r0 + j) * nseg + s]);
    const float best = row_max(bv);
    bi = row_min(bv == best ? bi : 0x7fffffff);
    if (gl == 0 && j < k) {
      if (row_argmax) row_argmax[r0 + j] = bi;
      if (!done && ((j == k - 1) || (bi != input_tokens[r0 + j + 1]))) atomicMin(&s_first_bad, j);
    }
    __syncthreads();
    if (!done && s_first_bad < j0 + GE_ROWS) {       // decided in this batch: its owner publishes the bonus token
      if (gl == 0 && j == s_first_bad) s_bonus = bi;
      done = true;
      if (!row_argmax) break;                        // (uniform) nothing else is wanted from the later rows
    }
  }
  __syncthreads();
  if (threadIdx.x == 0) { accept_len[seq] = s_first_bad; bonus_token[seq] = s_bonus; }
}

// ---------------------------------------------------------------------------------------
// Sampling, pass 1: per (row, segment) the maximum and the sum of exponentials of the
// temperature-scaled target and draft logits.  part [rows][segments][4] doubles:
// (max_t, sum_t, max_d, sum_d) with sum = sum exp(x*invT - max).
// ---------------------------------------------------------------------------------------
// e^y for y <= 0.  e^y = 2^(y log2 e): the product is formed in two pieces, so that its rounding
// error (which grows with |y|) and the low part of log2 e enter as a first-order correction of
// the hardware exp2 (good to 1 ulp).  About a third of the instructions of the library expf,
// which is what the streaming passes below were spending their time on.
__device__ __forceinline__ float exp_neg(float y) {
  y = fmaxf(y, -104.f);                               // e^-104 is below the smallest normal float
  const float t = y * 1.44269502e+00f;
  float r = fmaf(y, 1.44269502e+00f, -t);             // rounding error of t, exactly
  r = fmaf(y, 1.92596299e-08f, r);                    // log2 e = 1.44269502 + 1.92596299e-8
  const float e = __builtin_amdgcn_exp2f(t);
  return fmaf(e, r * 0.693147182f, e);
}

// Sampling, pass 1: per (row, segment) the maximum of x / T and sum exp(x / T - max), for the
// target and the draft logits.  Both segments are requested up front and held in registers (one
// memory latency per work-group), the maximum is found first and the sum taken relative to it: the
// maximum's own term is 1 up to the rounding of the scaled maximum (scale and subtraction are one FMA)
// and every other term's rounding error (|y| 2^-23 of itself, y = x / T - max <= 0) is weighted by its
// small size, so the plain hardware exp2 is accurate enough for a normaliser that is compared at 1e-5.
//   grid (segments, rows); part [rows][segments][4] = (max_t, sum_t, max_d, sum_d)
//   NR = rounds of ACC_BLOCK * 8 logits that cover a segment (registers held: 8 NR for bf16)
template <typename T, int NR, bool SHORT>
__global__ __launch_bounds__(ACC_BLOCK) void softmax_stats_partial_kernel(
    const T* __restrict__ target, const T* __restrict__ draft, long long row_stride, int vocab, int seg_len,
    float inv_t, double* __restrict__ part) {
  constexpr int NW = ACC_BLOCK / FD_WAVE;
  __shared__ float s_max[2][NW]; __shared__ double s_sum[2][NW];
  const int seg = blockIdx.x, row = blockIdx.y, nseg = gridDim.x;
  const int e0 = seg * seg_len, e1 = min(vocab, e0 + min(seg_len, NR * ACC_BLOCK * 8));
  RowShare<T, NR, SHORT> ht(e0, e1), hd(e0, e1);
  ht.request(target + (long long)row * row_stride);
  hd.request(draft + (long long)row * row_stride);
  float mt = ht.max() * inv_t, md = hd.max() * inv_t;              // (1 / T > 0: rounding keeps the order)
  ht.again(); hd.again();
  mt = wave_max(mt); md = wave_max(md);
  if ((threadIdx.x & 63) == 0) { s_max[0][threadIdx.x >> 6] = mt; s_max[1][threadIdx.x >> 6] = md; }
  __syncthreads();
  float Mt = s_max[0][0], Md = s_max[1][0];
#pragma unroll
  for (int w = 1; w < NW; ++w) { Mt = fmaxf(Mt, s_max[0][w]); Md = fmaxf(Md, s_max[1][w]); }
  float st = 0.f, sd = 0.f;
  const float L2E = 1.44269502e+00f;
  if (Mt > -INFINITY) st = ht.sum([&](float x) { return __builtin_amdgcn_exp2f((x * inv_t - Mt) * L2E); });
  if (Md > -INFINITY) sd = hd.sum([&](float x) { return __builtin_amdgcn_exp2f((x * inv_t - Md) * L2E); });
  const double wt = wave_sum((double)st), wd = wave_sum((double)sd);
  if ((threadIdx.x & 63) == 0) { s_sum[0][threadIdx.x >> 6] = wt; s_sum[1][threadIdx.x >> 6] = wd; }
  __syncthreads();
  if (threadIdx.x == 0) {
    double tt = 0.0, td = 0.0;
#pragma unroll
    for (int w = 0; w < NW; ++w) { tt += s_sum[0][w]; td += s_sum[1][w]; }
    double* o = part + ((long long)row * nseg + seg) * 4;
    o[0] = (double)Mt; o[1] = tt; o[2] = (double)Md; o[3] = td;
  }
}

// ---------------------------------------------------------------------------------------
// Sampling, pass 2: grid (chunk groups, sequences).  Every work-group first repeats the
// (cheap) accept tests of its sequence to find the stopping row j*, then sums the bonus
// token's weights -- residual max(0,p-q), and p itself -- over its share of the
// vocabulary, one double per 512-token chunk (one wave, 8 tokens per lane).
//   decision [B][4] int: (stop row, rejected?, -, -) written by group 0
//   chunk_res, chunk_p [B][nchunks] doubles
// ---------------------------------------------------------------------------------------
constexpr int CHUNK_TOK = FD_WAVE * 8;   // 512 tokens per chunk

template <typename T>
__global__ __launch_bounds__(ACC_BLOCK) void accept_sample_weights_kernel(
    const T* __restrict__ target, const T* __restrict__ draft, long long row_stride, int vocab, float inv_t,
    const double* __restrict__ part, int nseg,
    const int* __restrict__ row_indptr, const int* __restrict__ input_tokens,
    const float* __restrict__ u_accept, int total_rows, int max_rows_per_seq, int nchunks,
    int* __restrict__ decision, double* __restrict__ row_stats /*[B][4]*/,
    double* __restrict__ chunk_res, double* __restrict__ chunk_p) {
  const int seq = blockIdx.y, grp = blockIdx.x, ngrp = gridDim.x;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  constexpr int NW = ACC_BLOCK / FD_WAVE;
  int r0 = clampi(row_indptr[seq], 0, total_rows);
  int k = clampi(row_indptr[seq + 1] - r0, 0, min(max_rows_per_seq, total_rows - r0));
  if (k == 0) { if (grp == 0 && threadIdx.x == 0) { decision[seq * 4] = -1; decision[seq * 4 + 1] = 0; } return; }

  // Accept tests: SG lanes per row merge that row's segment statistics, ROWS_AT_ONCE rows at a time
  // (every load of a batch is in flight together).  The statistics of a batch stay in LDS, so the
  // row the step stops at -- the first rejected draft, else the last row -- is at hand afterwards.
  constexpr int SG = 16, ROWS_AT_ONCE = ACC_BLOCK / SG;
  __shared__ int s_first_bad;
  __shared__ double s_rows[ROWS_AT_ONCE][4];
  __shared__ double s_stats[4];
  const int grp16 = threadIdx.x / SG, gl = threadIdx.x % SG;
  if (threadIdx.x == 0) s_first_bad = k - 1;
  __syncthreads();
  int stop = k - 1;
  for (int j0 = 0; j0 < k; j0 += ROWS_AT_ONCE) {
    const int j = min(j0 + grp16, k - 1);                          // surplus lane groups repeat the last row
    const double* pr = part + (long long)(r0 + j) * nseg * 4;
    // the row's draft, its two logits and uniform: requested before the statistics, which they do not depend on
    const int d = j < k - 1 ? input_tokens[r0 + j + 1] : -1;         // the last row has no draft to test
    const bool d_ok = d >= 0 && d < vocab;
    float xt_d = 0.f, xd_d = 0.f, u_d = 0.f;
    if (d_ok) {
      xt_d = Elem<T>::load(target + (long long)(r0 + j) * row_stride + d);
      xd_d = Elem<T>::load(draft + (long long)(r0 + j) * row_stride + d);
      u_d = u_accept[r0 + j];
    }
    // a lane's first HELD segments are requested together and kept (4 pairs of rows 13.7 -> 12.7 us a call)
    constexpr int HELD = 4;
    typedef __attribute__((ext_vector_type(4))) double f64x4;
    f64x4 st[HELD];
#pragma unroll
    for (int u = 0; u < HELD; ++u) st[u] = *reinterpret_cast<const f64x4*>(pr + min(gl + u * SG, nseg - 1) * 4);
    double mt = -INFINITY, md = -INFINITY;
#pragma unroll
    for (int u = 0; u < HELD; ++u) {               // (the last segment repeated: no matter for a maximum)
      mt = fmax(mt, st[u][0]); md = fmax(md, st[u][2]);
      if (gl + u * SG >= nseg) st[u][1] = st[u][3] = 0.0;
    }
    for (int sg = gl + HELD * SG; sg < nseg; sg += SG) { mt = fmax(mt, pr[sg * 4]); md = fmax(md, pr[sg * 4 + 2]); }
    mt = row_max(mt); md = row_max(md);
    double zt = 0.0, zd = 0.0;
#pragma unroll
    for (int u = 0; u < HELD; ++u) {
      if (st[u][1] > 0.0) zt += st[u][1] * (double)exp_neg((float)(st[u][0] - mt));
      if (st[u][3] > 0.0) zd += st[u][3] * (double)exp_neg((float)(st[u][2] - md));
    }
    for (int sg = gl + HELD * SG; sg < nseg; sg += SG) {
      const double m0 = pr[sg * 4], s0 = pr[sg * 4 + 1], m1 = pr[sg * 4 + 2], s1 = pr[sg * 4 + 3];
      if (s0 > 0.0) zt += s0 * (double)exp_neg((float)(m0 - mt));     // maxima are floats held in doubles: the difference is exact
      if (s1 > 0.0) zd += s1 * (double)exp_neg((float)(m1 - md));
    }
    zt = row_sum(zt); zd = row_sum(zd);
    if (gl == 0 && j0 + grp16 < k) {
      s_rows[grp16][0] = mt; s_rows[grp16][1] = zt; s_rows[grp16][2] = md; s_rows[grp16][3] = zd;
      if (j < k - 1) {
        bool keep = false;
        if (d_ok) {
          const double p = (double)expf(xt_d * inv_t - (float)mt) / zt;
          const double q = (double)expf(xd_d * inv_t - (float)md) / zd;
          keep = (double)u_d * q < p;
        }
        if (!keep) atomicMin(&s_first_bad, j);
      }
    }
    __syncthreads();
    stop = s_first_bad;
    if (stop < j0 + ROWS_AT_ONCE) {                                 // the stopping row is in this batch
      if (threadIdx.x < 4) s_stats[threadIdx.x] = s_rows[stop - j0][threadIdx.x];
      break;                                                        // (uniform: every thread read the same stop)
    }
    __syncthreads();                                                // s_rows is rewritten by the next batch
  }
  __syncthreads();
  const bool rejected = stop < k - 1 ? true : false;   // stop == k-1 only when every draft was kept
  // (a rejection at row k-1 cannot happen: that row has no draft to test)
  const float Mt = (float)s_stats[0], Md = (float)s_stats[2];
  const double iZt = 1.0 / s_stats[1], iZd = 1.0 / s_stats[3];
  if (grp == 0 && threadIdx.x == 0) {
    decision[seq * 4] = stop; decision[seq * 4 + 1] = rejected ? 1 : 0;
    row_stats[seq * 4 + 0] = s_stats[0]; row_stats[seq * 4 + 1] = s_stats[1];
    row_stats[seq * 4 + 2] = s_stats[2]; row_stats[seq * 4 + 3] = s_stats[3];
  }
  const T* tp = target + (long long)(r0 + stop) * row_stride;
  const T* dp = draft + (long long)(r0 + stop) * row_stride;
  for (int c = grp * NW + wave; c < nchunks; c += ngrp * NW) {
    int e = c * CHUNK_TOK + lane * 8;
    double wres = 0.0, wp = 0.0;
    if (e < vocab) {
      float xt[8], xd[8];
      load_pair8(tp, dp, e, vocab, xt, xd);
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        double p = (double)expf(xt[i] * inv_t - Mt) * iZt;
        double q = (double)expf(xd[i] * inv_t - Md) * iZd;
        wp += p;
        wres += fmax(0.0, p - q);
      }
    }
    wres = wave_sum(wres); wp = wave_sum(wp);
    if (lane == 0) { chunk_res[(long long)seq * nchunks + c] = wres; chunk_p[(long long)seq * nchunks + c] = wp; }
  }
}

// ---------------------------------------------------------------------------------------
// Sampling, pass 3: one work-group per sequence.  Scan the chunk sums, find the chunk the
// scaled uniform falls into, then scan that chunk's 512 tokens with one wave.
// ---------------------------------------------------------------------------------------
template <typename T>
__global__ __launch_bounds__(ACC_BLOCK) void accept_sample_pick_kernel(
    const T* __restrict__ target, const T* __restrict__ draft, long long row_stride, int vocab, float inv_t,
    const int* __restrict__ row_indptr, const float* __restrict__ u_resample, int total_rows,
    int nchunks, const int* __restrict__ decision, const double* __restrict__ row_stats,
    const double* __restrict__ chunk_res, const double* __restrict__ chunk_p,
    int* __restrict__ accept_len, int* __restrict__ bonus_token) {
  const int seq = blockIdx.x;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  constexpr int NW = ACC_BLOCK / FD_WAVE;
  const int stop = decision[seq * 4];
  if (stop < 0) { if (threadIdx.x == 0) { accept_len[seq] = 0; bonus_token[seq] = -1; } return; }
  const int r0 = clampi(row_indptr[seq], 0, total_rows);
  const bool rejected = decision[seq * 4 + 1] != 0;
  __shared__ double s_wsum[NW];
  __shared__ int s_first;
  __shared__ int s_chunk; __shared__ double s_prefix;
  const double u = (double)u_resample[r0 + stop];
  const double st_mt = row_stats[seq * 4 + 0], st_zt = row_stats[seq * 4 + 1], st_md = row_stats[seq * 4 + 2], st_zd = row_stats[seq * 4 + 3];

  // Every thread takes a run of adjacent chunks; a scan over the 256 run sums gives each run what lies before it and the
  // total.  The first thread whose run crosses the scaled uniform walks its own chunks.  (One wave walking the chunks 64 at a
  // time, each batch loaded after the one before: 6.8 us for four sequences of 297 chunks, now 4.6.)
  const int per = (nchunks + ACC_BLOCK - 1) / ACC_BLOCK;
  const int c_lo = min((int)threadIdx.x * per, nchunks), c_hi = min(c_lo + per, nchunks);
  double own, ahead, W;
  auto scan = [&](const double* cw) {
    own = 0.0;
    for (int c = c_lo; c < c_hi; ++c) own += cw[c];
    const double inc = wave_prefix(own);
    if (lane == FD_WAVE - 1) s_wsum[wave] = inc;
    if (threadIdx.x == 0) s_first = ACC_BLOCK;
    __syncthreads();
    ahead = inc - own; W = 0.0;
#pragma unroll
    for (int w = 0; w < NW; ++w) { if (w < wave) ahead += s_wsum[w]; W += s_wsum[w]; }
  };
  const double* cw = (rejected ? chunk_res : chunk_p) + (long long)seq * nchunks;
  scan(cw);
  bool use_res = rejected;
  if (rejected && !(W > 0.0)) {                         // residual identically zero -> draw from p
    __syncthreads();
    use_res = false;
    cw = chunk_p + (long long)seq * nchunks;
    scan(cw);
  }
  const double thr = u * W;
  const bool hit = own > 0.0 && ahead + own > thr;
  const unsigned long long hits = __ballot(hit);
  if (hits && lane == __ffsll((long long)hits) - 1) atomicMin(&s_first, (int)threadIdx.x);
  __syncthreads();
  const int first = s_first;
  if ((int)threadIdx.x == (first < ACC_BLOCK ? first : 0)) {
    // (rounding corner: nobody crosses it, or the walk ends below it: the last chunk with weight)
    double run = first < ACC_BLOCK ? ahead : 0.0, pre = 0.0;
    int found = -1;
    const int from = first < ACC_BLOCK ? c_lo : 0, to = first < ACC_BLOCK ? c_hi : nchunks;
    for (int c = from; c < to; ++c) {
      const double w = cw[c];
      if (w > 0.0) { found = c; pre = run; }
      run += w;
      if (first < ACC_BLOCK && w > 0.0 && run > thr) break;
    }
    s_chunk = found < 0 ? 0 : found; s_prefix = pre;
  }
  __syncthreads();
  if (wave != 0) return;
  const int c = s_chunk;
  const float Mt = (float)st_mt, Md = (float)st_md;
  const double iZt = 1.0 / st_zt, iZd = 1.0 / st_zd;
  const T* tp = target + (long long)(r0 + stop) * row_stride;
  const T* dp = draft + (long long)(r0 + stop) * row_stride;
  const int e = c * CHUNK_TOK + lane * 8;
  double w8[8]; double lsum = 0.0;
#pragma unroll
  for (int i = 0; i < 8; ++i) w8[i] = 0.0;
  if (e < vocab) {
    float xt[8], xd[8];
    load_pair8(tp, dp, e, vocab, xt, xd);
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      double p = (double)expf(xt[i] * inv_t - Mt) * iZt;
      double q = (double)expf(xd[i] * inv_t - Md) * iZd;
      w8[i] = use_res ? fmax(0.0, p - q) : p;
      lsum += w8[i];
    }
  }
  const double inc = wave_prefix(lsum);
  double before = s_prefix + inc - lsum;
  int pick = -1;
  if (before + lsum > thr) {                            // the threshold is crossed inside this lane (or earlier)
    double run = before;
#pragma unroll
    for (int i = 0; i < 8; ++i) { run += w8[i]; if (pick < 0 && run > thr && w8[i] > 0.0) pick = e + i; }
  }
  unsigned long long m = __ballot(pick >= 0);
  int result;
  if (m) {
    result = __shfl(pick, __ffsll((long long)m) - 1);
  } else {                                              // rounding corner: last token of the chunk with weight
    int last = -1;
#pragma unroll
    for (int i = 0; i < 8; ++i) if (w8[i] > 0.0) last = e + i;
    unsigned long long m2 = __ballot(last >= 0);
    result = m2 ? __shfl(last, 63 - __clzll((long long)m2)) : min(vocab - 1, c * CHUNK_TOK);
  }
  if (lane == 0) { accept_len[seq] = stop; bonus_token[seq] = result; }
}

// ---------------------------------------------------------------------------------------
// Selective verification (Sec. 4.3, Eq. 5), pass 1: per (row, segment) of the drafter's logits the
// maximum, the lowest index holding it, and the sum of exp((x - max) / T) - the draft token and
// what its probability needs, in one pass with the segment held in registers.
//   grid (segments, rows); part_val/part_idx/part_sum [rows][segments]
// ---------------------------------------------------------------------------------------
template <typename T, int NR, bool SHORT>
__global__ __launch_bounds__(ACC_BLOCK) void draft_stats_partial_kernel(
    const T* __restrict__ logits, long long row_stride, int vocab, int seg_len, float inv_t,
    float* __restrict__ part_val, int* __restrict__ part_idx, double* __restrict__ part_sum) {
  const int seg = blockIdx.x, row = blockIdx.y, nseg = gridDim.x;
  const T* rp = logits + (long long)row * row_stride;
  const int e0 = seg * seg_len;
  RowShare<T, NR, SHORT> sh(e0, min(vocab, e0 + min(seg_len, NR * ACC_BLOCK * 8)));
  __shared__ float sv[ACC_BLOCK / FD_WAVE]; __shared__ int si[ACC_BLOCK / FD_WAVE];
  __shared__ double sd[ACC_BLOCK / FD_WAVE];
  sh.request(rp);
  const float m = sh.max();
  const float wm = wave_max(m);
  if ((threadIdx.x & 63) == 0) sv[threadIdx.x >> 6] = wm;
  __syncthreads();
  float M = sv[0];
#pragma unroll
  for (int w = 1; w < ACC_BLOCK / FD_WAVE; ++w) M = fmaxf(M, sv[w]);
  int bi = 0x7fffffff;
  float part = 0.f;
  sh.again();
  if (M > -INFINITY) {
    if (m == M) bi = sh.lowest_index_of(M);                  // few threads hold the maximum: only they look for it
    // The terms are summed relative to the segment's maximum, so the term of the maximum is exactly
    // 1 and every other term's rounding error (|y| * 2^-23 of itself, y = (x - M) / T <= 0) is
    // weighted by its own small size: the plain hardware exp2 is accurate enough here, and the pass
    // stays below the cost of the memory traffic.
    const float c = inv_t * 1.44269502e+00f;
    part = sh.sum([&](float x) { return __builtin_amdgcn_exp2f((x - M) * c); });
  }
  bi = wave_min(bi);
  const double ws = wave_sum((double)part);
  if ((threadIdx.x & 63) == 0) { si[threadIdx.x >> 6] = bi; sd[threadIdx.x >> 6] = ws; }
  __syncthreads();
  if (threadIdx.x == 0) {
    double tot = 0.0;
#pragma unroll
    for (int w = 0; w < ACC_BLOCK / FD_WAVE; ++w) { bi = min(bi, si[w]); tot += sd[w]; }
    const long long o = (long long)row * nseg + seg;
    part_val[o] = M; part_idx[o] = bi; part_sum[o] = tot;
  }
}

// ---------------------------------------------------------------------------------------
// Selective verification, pass 2: one work-group per sequence, DS_GROUP lanes per row, sixteen rows
// at a time.  A lane group merges its row's segments into the draft token and its probability
// p = 1 / sum_v exp((x_v - max) / T); thread 0 then walks the rows in order with the running
// product of the probabilities and counts the positions whose product is still at or above the
// threshold (Eq. 5); the first one below it ends the count.
// ---------------------------------------------------------------------------------------
constexpr int DS_GROUP = 16;
constexpr int DS_ROWS = ACC_BLOCK / DS_GROUP;
constexpr int DS_HELD = 4;

__global__ __launch_bounds__(ACC_BLOCK) void draft_select_epilogue_kernel(
    const float* __restrict__ part_val, const int* __restrict__ part_idx, const double* __restrict__ part_sum,
    int nseg, float inv_t, float threshold, const int* __restrict__ row_indptr, int total_rows, int max_rows_per_seq,
    int* __restrict__ draft_tokens, float* __restrict__ confidence, int* __restrict__ keep_len) {
  const int seq = blockIdx.x, grp = threadIdx.x / DS_GROUP, gl = threadIdx.x % DS_GROUP;
  const int r0 = clampi(row_indptr[seq], 0, total_rows);
  const int k = clampi(row_indptr[seq + 1] - r0, 0, min(max_rows_per_seq, total_rows - r0));
  __shared__ double s_p[DS_ROWS];
  double prod = 1.0;
  int keep = 0;
  bool open = true;
  for (int j0 = 0; j0 < k; j0 += DS_ROWS) {                  // k is uniform over the group
    const int j = min(j0 + grp, k - 1);                      // surplus lane groups repeat the last row, unwritten
    const long long base = (long long)(r0 + j) * nseg;
    // A lane's first DS_HELD segments (all of them up to 655360 logits a row) are requested together: their maxima first, the rest
    // when the row's maximum is known, was two latencies of memory (8 rows 8.4 -> 7.1 us a call, 480 rows 28.2 -> 27.8).
    float v[DS_HELD]; int ix[DS_HELD]; double sm[DS_HELD];
#pragma unroll
    for (int u = 0; u < DS_HELD; ++u) {
      const int s = min(gl + u * DS_GROUP, nseg - 1);
      v[u] = part_val[base + s]; ix[u] = part_idx[base + s]; sm[u] = part_sum[base + s];
    }
    float m = -INFINITY;
#pragma unroll
    for (int u = 0; u < DS_HELD; ++u) {
      if (gl + u * DS_GROUP >= nseg) v[u] = -INFINITY;
      m = fmaxf(m, v[u]);
    }
    for (int s = gl + DS_HELD * DS_GROUP; s < nseg; s += DS_GROUP) m = fmaxf(m, part_val[base + s]);
    m = row_max(m);
    int bi = 0x7fffffff; double z = 0.0;
#pragma unroll
    for (int u = 0; u < DS_HELD; ++u) {
      if (v[u] == m && gl + u * DS_GROUP < nseg) bi = min(bi, ix[u]);
      if (v[u] > -INFINITY) z += sm[u] * (double)exp_neg((v[u] - m) * inv_t);
    }
    for (int s = gl + DS_HELD * DS_GROUP; s < nseg; s += DS_GROUP) {
      const float w = part_val[base + s];
      if (w == m) bi = min(bi, part_idx[base + s]);
      if (w > -INFINITY) z += part_sum[base + s] * (double)exp_neg((w - m) * inv_t);
    }
    bi = row_min(bi);
    z = row_sum(z);
    const double pj = z > 0.0 ? 1.0 / z : 0.0;
    if (gl == 0 && j0 + grp < k) {
      draft_tokens[r0 + j] = bi == 0x7fffffff ? -1 : bi;
      if (confidence) confidence[r0 + j] = (float)pj;
      s_p[grp] = pj;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
      const int nrow = min(DS_ROWS, k - j0);
      for (int i = 0; i < nrow; ++i) {
        prod *= s_p[i];
        if (open && prod >= (double)threshold) ++keep; else open = false;
      }
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) keep_len[seq] = keep;
}

// ---------------------------------------------------------------------------------------
// Branch selection (Sec. 3, parallel speculative decoding): one wave per sequence copies the
// block drafted under the number of accepted drafts that verification arrived at.
// ---------------------------------------------------------------------------------------
__global__ __launch_bounds__(FD_WAVE) void select_branch_kernel(
    const int* __restrict__ block_tokens, const int* __restrict__ block_indptr, const int* __restrict__ mask_blocks,
    const int* __restrict__ accept_len, const int* __restrict__ first_vis, const int* __restrict__ verify_len,
    int total_tokens, int out_stride, int* __restrict__ out_tokens, int* __restrict__ out_block) {
  const int seq = blockIdx.x, lane = threadIdx.x;
  const int t0 = clampi(block_indptr[seq], 0, total_tokens);
  const int len = clampi(block_indptr[seq + 1] - t0, 0, total_tokens - t0);
  const int nb = mask_blocks[seq];
  int* o = out_tokens + (long long)seq * out_stride;
  const bool ok = nb >= 1 && len % (nb >= 1 ? nb : 1) == 0 && len / (nb >= 1 ? nb : 1) <= out_stride;
  const int mb = ok ? len / nb : 0;
  int b = -1;
  if (ok) {
    // without first_vis: the attention call's own default, the last block sees every verify row
    const int fv = first_vis ? first_vis[seq] : max(verify_len[seq] - nb + 1, 0);
    b = accept_len[seq] + 1 - fv;
    b = clampi(b, 0, nb - 1);
  }
  for (int j = lane; j < out_stride; j += FD_WAVE) o[j] = j < mb ? block_tokens[t0 + b * mb + j] : -1;
  if (out_block && lane == 0) out_block[seq] = b;
}

hipError_t run_select_branch(const int* block_tokens, const int* block_indptr, const int* mask_blocks,
                             const int* accept_len, const int* first_vis, const int* verify_len, int batch,
                             int total_tokens, int out_stride, int* out_tokens, int* out_block, hipStream_t st) {
  hipLaunchKernelGGL(select_branch_kernel, dim3(batch), dim3(FD_WAVE), 0, st, block_tokens, block_indptr,
                     mask_blocks, accept_len, first_vis, verify_len, total_tokens, out_stride, out_tokens, out_block);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------------------
// host-side launchers (called from api.hip)
// ---------------------------------------------------------------------------------------
static inline int pick_segments(int rows, int vocab) {
  // Around 2048 work-groups in all, each taking a whole number of rounds (ACC_BLOCK * 8 logits, one
  // 16-byte load per lane): at least two rounds, so that a group has 4096 logits to work on, and
  // never more than the passes hold in registers.
  int want = (2048 + rows - 1) / (rows > 0 ? rows : 1);
  if (want < 1) want = 1;
  if (want > 64) want = 64;
  const long long round_len = (long long)ACC_BLOCK * 8;
  long long r = (vocab + want * round_len - 1) / (want * round_len);
  if (r < 2) r = 2;
  if (r > ARG_ROUNDS) r = ARG_ROUNDS;
  long long s = (vocab + r * round_len - 1) / (r * round_len);
  return (int)(s < 1 ? 1 : s);
}
static inline int seg_len_for(int vocab, int nseg) {
  int l = (vocab + nseg - 1) / nseg;
  return (l + 7) / 8 * 8;
}

// The kernel variant for segments of seg_len logits: as many rounds of ACC_BLOCK * 8 logits as cover a segment (<= ARG_ROUNDS); rows of fewer
// than eight logits have one of their own.  A round beyond the segment's end costs the arithmetic of one that is not (always
// five rounds / as many as needed, us a call, bf16 rows of 151936: selection over 8 rows 7.1 / 5.9, over 64 11.2 / 9.1; greedy acceptance of 8
// rows 6.0 / 5.5, of 32 rows of floats 9.4 / 8.5; from 128 rows on five are needed).
template <typename F> static void with_rounds(int seg_len, int vocab, F&& launch) {
  if (vocab < 8) { launch(std::integral_constant<int, 1>{}, std::true_type{}); return; }
  switch ((seg_len + ACC_BLOCK * 8 - 1) / (ACC_BLOCK * 8)) {
    case 1: launch(std::integral_constant<int, 1>{}, std::false_type{}); break;
    case 2: launch(std::integral_constant<int, 2>{}, std::false_type{}); break;
    case 3: launch(std::integral_constant<int, 3>{}, std::false_type{}); break;
    case 4: launch(std::integral_constant<int, 4>{}, std::false_type{}); break;
    default: launch(std::integral_constant<int, ARG_ROUNDS>{}, std::false_type{}); break;
  }
}

// Sampling workspace layout (all blocks 256-byte aligned), shared by the size query and the launcher.
struct SampleLayout {
  size_t part, row_stats, chunk_res, chunk_p, decision, total;
  int nseg, nchunks;
};
static inline size_t align256(size_t x) { return (x + 255) / 256 * 256; }
static inline SampleLayout sample_layout(int batch, int total_rows, int vocab) {
  SampleLayout l;
  size_t rows = (size_t)(total_rows > 0 ? total_rows : 1), seqs = (size_t)(batch > 0 ? batch : 1);
  l.nseg = pick_segments(total_rows, vocab);
  l.nchunks = (vocab + CHUNK_TOK - 1) / CHUNK_TOK;
  size_t off = 0;
  l.part = off;      off += align256(rows * l.nseg * 4 * sizeof(double));
  l.row_stats = off; off += align256(seqs * 4 * sizeof(double));
  l.chunk_res = off; off += align256(seqs * l.nchunks * sizeof(double));
  l.chunk_p = off;   off += align256(seqs * l.nchunks * sizeof(double));
  l.decision = off;  off += align256(seqs * 4 * sizeof(int));
  l.total = off;
  return l;
}

size_t accept_workspace_bytes(int batch, int total_rows, int vocab, int sampling) {
  if (batch < 0 || total_rows < 0 || vocab <= 0) return 0;
  if (sampling) return sample_layout(batch, total_rows, vocab).total;
  size_t rows = (size_t)(total_rows > 0 ? total_rows : 1);
  return align256(rows * pick_segments(total_rows, vocab) * (sizeof(float) + sizeof(int)));
}

template <typename T>
static hipError_t launch_greedy(const T* logits, long long row_stride, int vocab, const int* row_indptr,
                                const int* toks, int batch, int total_rows, int max_rows, int* accept_len,
                                int* bonus, int* row_argmax, void* ws, hipStream_t st) {
  int nseg = pick_segments(total_rows, vocab);
  int sl = seg_len_for(vocab, nseg);
  float* pv = reinterpret_cast<float*>(ws);
  int* pi = reinterpret_cast<int*>(pv + (size_t)(total_rows > 0 ? total_rows : 1) * nseg);
  if (total_rows > 0)
    with_rounds(sl, vocab, [&](auto nr, auto is_short) {
      hipLaunchKernelGGL((argmax_partial_kernel<T, decltype(nr)::value, decltype(is_short)::value>), dim3(nseg, total_rows), dim3(ACC_BLOCK), 0, st,
                         logits, row_stride, vocab, sl, pv, pi);
    });
  if (batch > 0)
    hipLaunchKernelGGL(accept_greedy_epilogue_kernel, dim3(batch), dim3(ACC_BLOCK), 0, st,
                       pv, pi, nseg, row_indptr, toks, total_rows, max_rows, accept_len, bonus, row_argmax);
  return hipGetLastError();
}

template <typename T>
static hipError_t launch_sample(const T* target, const T* draft, long long row_stride, int vocab, float temperature,
                                const int* row_indptr, const int* toks, const float* ua, const float* ur,
                                int batch, int total_rows, int max_rows, int* accept_len, int* bonus,
                                void* ws, hipStream_t st) {
  const SampleLayout lay = sample_layout(batch, total_rows, vocab);
  const int nseg = lay.nseg, nchunks = lay.nchunks;
  const int sl = seg_len_for(vocab, nseg);
  char* base = reinterpret_cast<char*>(ws);
  double* part = reinterpret_cast<double*>(base + lay.part);
  double* row_stats = reinterpret_cast<double*>(base + lay.row_stats);
  double* chunk_res = reinterpret_cast<double*>(base + lay.chunk_res);
  double* chunk_p = reinterpret_cast<double*>(base + lay.chunk_p);
  int* decision = reinterpret_cast<int*>(base + lay.decision);
  float inv_t = 1.0f / temperature;
  if (total_rows > 0)
    with_rounds(sl, vocab, [&](auto nr, auto is_short) {
      hipLaunchKernelGGL((softmax_stats_partial_kernel<T, decltype(nr)::value, decltype(is_short)::value>), dim3(nseg, total_rows), dim3(ACC_BLOCK), 0, st,
                         target, draft, row_stride, vocab, sl, inv_t, part);
    });
  if (batch > 0) {
    int groups = (nchunks + (ACC_BLOCK / FD_WAVE) - 1) / (ACC_BLOCK / FD_WAVE);
    int want = (1024 + batch - 1) / batch;
    if (groups > want) groups = want;
    if (groups < 1) groups = 1;
    hipLaunchKernelGGL(accept_sample_weights_kernel<T>, dim3(groups, batch), dim3(ACC_BLOCK), 0, st,
                       target, draft, row_stride, vocab, inv_t, part, nseg, row_indptr, toks, ua,
                       total_rows, max_rows, nchunks, decision, row_stats, chunk_res, chunk_p);
    hipLaunchKernelGGL(accept_sample_pick_kernel<T>, dim3(batch), dim3(ACC_BLOCK), 0, st,
                       target, draft, row_stride, vocab, inv_t, row_indptr, ur, total_rows, nchunks,
                       decision, row_stats, chunk_res, chunk_p, accept_len, bonus);
  }
  return hipGetLastError();
}

size_t draft_select_workspace_bytes(int total_rows, int vocab) {
  const size_t slots = (size_t)(total_rows > 0 ? total_rows : 1) * pick_segments(total_rows, vocab);
  return align256(slots * sizeof(float)) + align256(slots * sizeof(int)) + align256(slots * sizeof(double));
}

template <typename T>
static hipError_t launch_draft_select(const T* logits, long long row_stride, int vocab, float temperature, float threshold,
                                      const int* row_indptr, int batch, int total_rows, int max_rows, int* tokens,
                                      float* confidence, int* keep_len, void* ws, hipStream_t st) {
  const int nseg = pick_segments(total_rows, vocab);
  const int sl = seg_len_for(vocab, nseg);
  const size_t slots = (size_t)(total_rows > 0 ? total_rows : 1) * nseg;
  char* base = reinterpret_cast<char*>(ws);
  float* pv = reinterpret_cast<float*>(base);
  int* pi = reinterpret_cast<int*>(base + align256(slots * sizeof(float)));
  double* pd = reinterpret_cast<double*>(base + align256(slots * sizeof(float)) + align256(slots * sizeof(int)));
  const float inv_t = 1.0f / temperature;
  if (total_rows > 0)
    with_rounds(sl, vocab, [&](auto nr, auto is_short) {
      hipLaunchKernelGGL((draft_stats_partial_kernel<T, decltype(nr)::value, decltype(is_short)::value>), dim3(nseg, total_rows), dim3(ACC_BLOCK), 0, st,
                         logits, row_stride, vocab, sl, inv_t, pv, pi, pd);
    });
  if (batch > 0)
    hipLaunchKernelGGL(draft_select_epilogue_kernel, dim3(batch), dim3(ACC_BLOCK), 0, st, pv, pi, pd, nseg, inv_t,
                       threshold, row_indptr, total_rows, max_rows, tokens, confidence, keep_len);
  return hipGetLastError();
}

hipError_t run_draft_select(const void* logits, int dt, long long row_stride, int vocab, float temperature,
                            float threshold, const int* row_indptr, int batch, int total_rows, int max_rows,
                            int* tokens, float* confidence, int* keep_len, void* ws, hipStream_t st) {
  if (dt == FD_BF16)
    return launch_draft_select<bf16_t>((const bf16_t*)logits, row_stride, vocab, temperature, threshold, row_indptr,
                                       batch, total_rows, max_rows, tokens, confidence, keep_len, ws, st);
  return launch_draft_select<float>((const float*)logits, row_stride, vocab, temperature, threshold, row_indptr,
                                    batch, total_rows, max_rows, tokens, confidence, keep_len, ws, st);
}

hipError_t run_accept_greedy(const void* logits, int dt, long long row_stride, int vocab, const int* row_indptr,
                             const int* toks, int batch, int total_rows, int max_rows, int* accept_len,
                             int* bonus, int* row_argmax, void* ws, hipStream_t st) {
  if (dt == FD_BF16)
    return launch_greedy<bf16_t>((const bf16_t*)logits, row_stride, vocab, row_indptr, toks, batch, total_rows,
                                 max_rows, accept_len, bonus, row_argmax, ws, st);
  return launch_greedy<float>((const float*)logits, row_stride, vocab, row_indptr, toks, batch, total_rows,
                              max_rows, accept_len, bonus, row_argmax, ws, st);
}

hipError_t run_accept_sample(const void* target, const void* draft, int dt, long long row_stride, int vocab,
                             float temperature, const int* row_indptr, const int* toks, const float* ua,
                             const float* ur, int batch, int total_rows, int max_rows, int* accept_len,
                             int* bonus, void* ws, hipStream_t st) {
  if (dt == FD_BF16)
    return launch_sample<bf16_t>((const bf16_t*)target, (const bf16_t*)draft, row_stride, vocab, temperature,
                                 row_indptr, toks, ua, ur, batch, total_rows, max_rows, accept_len, bonus, ws, st);
  return launch_sample<float>((const float*)target, (const float*)draft, row_stride, vocab, temperature,
                              row_indptr, toks, ua, ur, batch, total_rows, max_rows, accept_len, bonus, ws, st);
}

}  // namespace fd
