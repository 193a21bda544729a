// Long overlap-save transforms (N = 2^15 .. 2^26 complex points) as a four-step FFT.
//
// The paper dedisperses the full band with transforms of millions of points
// (Sec. 1.3, 2.3, 4.5); here N = N1 * N2 with n = n1 + N1 n2 and
// k = k2 + N2 k1:
//   cols_fwd : for each column n1, DFT over n2 of x[n1 + N1 n2] (length N2),
//              times W_N^(n1 k2), stored row-major as S[k2][n1]
//   rows     : for each row k2, DFT over n1 (length N1) gives X[k2 + N2 k1];
//              multiply by the chirp of Eq. 3 (and 1/N); inverse DFT over k1;
//              times W_N^(-n1 k2); stored back in place as S[k2][n1]
//   cols_inv : for each column n1, inverse DFT over k2 gives z[n1 + N1 n2];
//              samples [nfront, nfront + M) of block k become y[k M + m]:
//              |y|^2 to a per-sample buffer and, if asked, y itself
//   integrate: P[u] = sum of n_int consecutive |y|^2
// Above 2^22 points (N2 > 2048) each column transform is itself split in
// two, N2 = A B with n2 = a + A b and k2 = kb + B ka, so the column passes
// become two passes each (see "Three-level transforms" below); the spectrum
// bin k2 of a block is then stored in row ka + A kb.
// Every sub-transform reuses the register/LDS Stockham passes of the block
// kernel; a workgroup runs G sub-transforms side by side, lanes ordered so
// that global accesses along n1 are contiguous.  The twiddles W_N^(n1 k2)
// are computed (exact phase in turns, hardware sine and cosine), not read
// from a table.  The same passes carry the full-band mode (further below):
// a real series packed two samples per complex value, the row pass holding
// the mirror rows of each bin pair.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <string>
#include <type_traits>
#include <vector>

#include "cdd_fft.h"
#include "cdd_fullband.h"
#include "cdd_internal.h"

namespace cdd {

// Sub-transform schedules (length L, Tsub threads, 16 points per thread).
// Twiddles are loaded ahead of the exchange before the pass that takes them: one
// channel of 2^23 samples at 2^18 points (1024 x 256) 138 -> 131 us, of 2^25 samples
// 466 -> 446 us; not at 512 and 2048 points, where the registers cost as much as
// the wait (2^20 points 331 -> 341 us with both).
template <int L>
struct SubSched;
template <> struct SubSched<128> { using type = Sched<128, 8, 8, 16, 1, 1, true, true>; };
template <> struct SubSched<256> { using type = Sched<256, 16, 16, 16, 1, 1, true, true>; };
template <> struct SubSched<512> { using type = Sched<512, 32, 8, 8, 8, 1>; };
template <> struct SubSched<1024> { using type = Sched<1024, 64, 16, 16, 4, 1, true, true>; };
template <> struct SubSched<2048> { using type = Sched<2048, 128, 16, 16, 8, 1>; };

struct LargeArgs {
  const void* x;        // channel-major input [nchan][nsamp]
  float2* S;            // [items][N] intermediate spectra (items of this chunk)
  float* p;             // [nchan][nsamp] |y|^2
  float2* vout;         // [nchan][nsamp] or null
  const float2* twc;    // column sub-transform twiddles
  const float2* twr;    // row sub-transform twiddles
  int64_t nsamp, nblocks, item0;
  int32_t nchan, N1, N2, M, nfront, phase_mode, exact_div, taper;
  double f_lo, df, dconst, dm;
  // full-band mode: Eq. 3's phase at bin j is qb j^2 / (1 + qbeta j) turns; the
  // chirp function per real-spectrum bin (N + 1 entries), or null to form it in
  // the row pass
  double qb, qbeta;
  const float2* hb;
  int32_t lgn, lg1;  // log2(N1 N2), log2(N1)
  float gain;        // relative correction of the transforms' gain (split_gain)
  // fused detection + integration in cols_inv (n_int divides the G columns
  // of a workgroup): P and the t_int outputs per channel, and the partial
  // sums of the groups that straddle two column runs (in p: per item, two
  // per run of G samples)
  float* P;
  int64_t t_int;
  int32_t n_int;
  int32_t fuse;
  // three-level transforms: N2 = A B (A = 1 for the two-level form), the
  // twiddles of the length-A sub-transform, and log2 of N2 and B
  int32_t A, lg2, lgB;
  // three-level transforms: the column classes kb of this launch of the middle
  // and row passes (see run_passes): un of them from u0, in the full-band mode
  // with their mirror classes (see mirror_class)
  int32_t u0, un;
  const float2* twm;
  // one-channel calls: coverage set to 1 by the chirp-table kernel (or null)
  int32_t* cov_fill;
  int64_t cov_n;
};

// Row of the intermediate array that holds spectrum bin k2 (< N2): k2 itself
// in the two-level form; ka + A kb for k2 = kb + B ka in the three-level one.
__device__ __forceinline__ int64_t spec_row(const LargeArgs& a, int k2) {
  if (a.A == 1) return k2;
  return (int64_t)(k2 >> a.lgB) + (int64_t)a.A * (k2 & ((1 << a.lgB) - 1));
}

// Byte offsets into one item's spectra or samples fit 32 bits (N 8 <= 2^29), so
// the passes address them through a buffer resource on the item's base: one
// vector offset per thread and scalar offsets per element, where 64-bit
// addresses took two to four vector operations each.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t item_rsrc(const void* base, int64_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc((void*)base, (short)0, (int)bytes, 0x00020000);
}
typedef unsigned int uint2v __attribute__((ext_vector_type(2)));
__device__ __forceinline__ float2 bload2(__amdgpu_buffer_rsrc_t rs, int voff, int soff) {
  return __builtin_bit_cast(float2, __builtin_amdgcn_raw_buffer_load_b64(rs, voff, soff, 0));
}
__device__ __forceinline__ void bstore2(__amdgpu_buffer_rsrc_t rs, float2 v, int voff, int soff) {
  __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(uint2v, v), rs, voff, soff, 0);
}

// exp(-2 pi i v / 2^32): v is a phase shifted up so that its turn fills 32
// bits (m << (32 - lg) for m / 2^lg turns; whole turns fall off the top, so
// products and sums may wrap).  Read as a signed number it lies in [-1/2, 1/2)
// turn, and its conversion to FP32 is the only rounding (none up to lg = 24,
// correctly rounded beyond).
__device__ __forceinline__ float2 expi_phase(uint32_t v) {
  const float t = (float)(int32_t)v * 0x1p-32f;
  return make_float2(__builtin_amdgcn_cosf(t), -__builtin_amdgcn_sinf(t));
}

// The four-step twiddles W_N^(n1 k2) are formed this way (the hardware sine and
// cosine take turns; absolute error about 1.2e-7) rather than read from a
// table, whose scattered indices (n1 k2) touch a cache line per lane.

// ---------------------------------------------------------------------------
// cols_fwd
// ---------------------------------------------------------------------------
// Two-level form (THREE = false): the length-N2 column transforms.  Three-
// level form: the length-B transforms over b of x[n1 + N1 (a + A b)] for
// each a, times W_N2^(a kb), stored in row a + A kb (the first half of the
// column transform; cols_mid_kernel does the second).
template <class SC, int G, int DT, bool THREE>
__global__ __launch_bounds__(SC::T * G) void cols_fwd_kernel(const LargeArgs a) {
  __shared__ float lds[G * (SC::lds_floats() + 1)];
  constexpr int L = SC::N, R0 = SC::rad_f(0), B0 = L / (R0 * SC::T);
  constexpr int RL = SC::rad_f(SC::NP - 1), BL = L / (RL * SC::T);
  const int t = threadIdx.x, g = t % G, tl = t / G;
  const int ngrp = a.N1 / G;
  const int nsub = THREE ? a.A : 1;
  const int64_t item = a.item0 + blockIdx.x / ((unsigned)ngrp * nsub);
  const int rem = (int)(blockIdx.x % ((unsigned)ngrp * nsub));
  const int sa = THREE ? rem / ngrp : 0;  // a of this column run
  const int n1 = (rem % ngrp) * G + g;
  const int c = (int)(item / a.nblocks);
  const int64_t k = item - (int64_t)c * a.nblocks;
  constexpr int ES = DT == CDD_CI8 ? 2 : 8;
  const int64_t start = k * a.M - a.nfront;
  const int pitch = THREE ? a.N1 * a.A : a.N1;  // samples between successive l (n2 = sa + A l)
  const int v0 = n1 + a.N1 * sa + tl * pitch;
  float2 v[SC::E];
  if (start >= 0) {
    // the resource ends at the data's end: the hardware returns zeros past it
    const int64_t avail = a.nsamp - start, N = (int64_t)a.N1 * a.N2;
    const __amdgpu_buffer_rsrc_t rs =
        item_rsrc((const char*)a.x + ((int64_t)c * a.nsamp + start) * ES,
                  (avail < N ? (avail > 0 ? avail : 0) : N) * ES);
#pragma unroll
    for (int b = 0; b < B0; ++b)
#pragma unroll
      for (int r = 0; r < R0; ++r) {
        const int soff = (SC::T * b + r * (L / R0)) * pitch * ES;
        if constexpr (DT == CDD_CI8) {
          const unsigned short w = __builtin_amdgcn_raw_buffer_load_b16(rs, v0 * ES, soff, 0);
          v[b * R0 + r] = make_float2((float)(signed char)(w & 0xff), (float)(signed char)(w >> 8));
        } else {
          v[b * R0 + r] = bload2(rs, v0 * ES, soff);
        }
      }
  } else {
#pragma unroll
    for (int b = 0; b < B0; ++b)
#pragma unroll
      for (int r = 0; r < R0; ++r) {
        const int64_t ts = start + v0 + (SC::T * b + r * (L / R0)) * pitch;
        float2 z = make_float2(0.f, 0.f);
        if (ts >= 0 && ts < a.nsamp) {
          if constexpr (DT == CDD_CI8) {
            const short w = ((const short*)a.x)[(int64_t)c * a.nsamp + ts];
            z = make_float2((float)(signed char)(w & 0xff), (float)(signed char)(w >> 8));
          } else {
            z = ((const float2*)a.x)[(int64_t)c * a.nsamp + ts];
          }
        }
        v[b * R0 + r] = z;
      }
  }
  fft_forward<SC>(v, lds + g * (SC::lds_floats() + 1), a.twc, tl);
  const int64_t N = (int64_t)a.N1 * a.N2;
  const __amdgpu_buffer_rsrc_t so = item_rsrc(a.S + (item - a.item0) * N, N * 8);
  // output kk goes to row kk (sa + A kk) times the twiddle of n1 kk / N (sa kk / N2)
  const uint32_t ph = THREE ? (uint32_t)sa << (32 - a.lg2) : (uint32_t)n1 << (32 - a.lgn);
#pragma unroll
  for (int b = 0; b < BL; ++b)
#pragma unroll
    for (int r = 0; r < RL; ++r) {
      const int kc = SC::T * b + r * (L / RL);
      bstore2(so, cmul(v[b * RL + r], expi_phase(ph * (uint32_t)(tl + kc))), v0 * 8,
              kc * pitch * 8);
    }
}

// ---------------------------------------------------------------------------
// Three-level transforms: the second half of each column transform.  With
// n2 = a + A b and k2 = kb + B ka, the length-N2 column DFT is
//   C[kb + B ka] = sum_a W_A^(a ka) W_N2^(a kb) sum_b x[a + A b] W_B^(b kb);
// cols_fwd_kernel forms the inner sums (times W_N2^(a kb)) in rows a + A kb,
// and this kernel, for each kb, the outer sums over a, times the four-step
// twiddle W_N^(n1 k2), back into the same rows (bin k2 in row ka + A kb).
// The inverse (INV) takes the same steps backwards: the inverse DFT over ka
// of rows ka + A kb, times W_N2^(-a kb), into rows a + A kb, before
// cols_inv_kernel's inverse DFTs over kb.
// ---------------------------------------------------------------------------
// Class m of the full-band mode's launches: classes 2j and 2j + 1 are a mirror
// pair (kb, B - kb), the first pair the two classes that mirror themselves.
__device__ __forceinline__ int mirror_class(const LargeArgs& a, int m) {
  const int B = 1 << a.lgB, j = m >> 1;
  return j == 0 ? (m & 1) * (B / 2) : m & 1 ? B - j : j;
}

template <class SC, int G, bool INV, bool REAL>
__global__ __launch_bounds__(SC::T * G) void cols_mid_kernel(const LargeArgs a) {
  __shared__ float lds[G * (SC::lds_floats() + 1)];
  constexpr int L = SC::N;  // A
  constexpr int RIN = INV ? SC::rad_i(0) : SC::rad_f(0), BIN = L / (RIN * SC::T);
  constexpr int ROUT = INV ? SC::rad_f(0) : SC::rad_f(SC::NP - 1), BOUT = L / (ROUT * SC::T);
  const int t = threadIdx.x, g = t % G, tl = t / G;
  const int ngrp = a.N1 / G;
  const int nsub = REAL ? 2 * a.un : a.un;
  const int64_t item = a.item0 + blockIdx.x / ((unsigned)ngrp * nsub);
  const int rem = (int)(blockIdx.x % ((unsigned)ngrp * nsub));
  const int kb = REAL ? mirror_class(a, 2 * a.u0 + rem / ngrp) : a.u0 + rem / ngrp;
  const int n1 = (rem % ngrp) * G + g;
  // rows l + A kb (l < A) of this item, column n1
  const __amdgpu_buffer_rsrc_t rs = item_rsrc(
      a.S + (item - a.item0) * ((int64_t)a.N1 * a.N2) + (int64_t)L * kb * a.N1,
      (int64_t)L * a.N1 * 8);
  const int voff = (n1 + tl * a.N1) * 8, pitch = a.N1 * 8;
  float2 v[SC::E];
#pragma unroll
  for (int b = 0; b < BIN; ++b)
#pragma unroll
    for (int r = 0; r < RIN; ++r)
      v[b * RIN + r] = bload2(rs, voff, (SC::T * b + r * (L / RIN)) * pitch);
  float* my = lds + g * (SC::lds_floats() + 1);
  if (INV)
    fft_inverse<SC>(v, my, a.twm, tl);
  else
    fft_forward<SC>(v, my, a.twm, tl);
  // twiddle of kk kb / N2 (conjugate), or of n1 (kb + B kk) / N
  const uint32_t ph = INV ? (uint32_t)kb << (32 - a.lg2) : (uint32_t)n1 << (32 - a.lgn);
#pragma unroll
  for (int b = 0; b < BOUT; ++b)
#pragma unroll
    for (int r = 0; r < ROUT; ++r) {
      const int kc = SC::T * b + r * (L / ROUT);
      const uint32_t kk = (uint32_t)(tl + kc);
      float2 w = expi_phase(ph * (INV ? kk : (uint32_t)kb + (kk << a.lgB)));
      if (INV) w.y = -w.y;
      bstore2(rs, cmul(v[b * ROUT + r], w), voff, kc * pitch);
    }
}

// ---------------------------------------------------------------------------
// Chirp function of channel c at bin i of the N-point transform (bin i < N/2
// lies +i df/N from the channel centre, else (i - N) df/N): exp(-2 pi i q) of
// Eq. 3 about the centre, times the taper and 1/N.  FP64 phase reduced before
// the FP32 rotation, or all FP32 (precision study).
// ---------------------------------------------------------------------------
__device__ __forceinline__ float2 chan_chirp(const LargeArgs& a, double fc, int64_t i,
                                             int64_t N) {
  const float inv_n = 1.0f / (float)N;
  const int64_t si = i < N / 2 ? i : i - N;
  const float g = inv_n * taper_gain<false>(a.taper, (float)si * inv_n);
  if (a.phase_mode == CDD_PHASE_FP64_REDUCED) {
    const double dfn = a.df / (double)N;
    const double B = a.dconst * a.dm * dfn * dfn / (fc * fc * fc);
    const double beta = dfn / fc;
    const double sd = (double)si;
    const double x = beta * sd;
    const double q = a.exact_div ? (B * (sd * sd)) / fma(beta, sd, 1.0)
                                 : (B * (sd * sd)) * fma(x, x, 1.0 - x);
    const float2 h = expi_neg_turns_fp32(q - rint(q), RotationSize{1.0f, a.gain});
    return make_float2(h.x * g, h.y * g);
  }
  const float fcf = (float)fc;
  const float Af = (float)(a.dconst * a.dm) / (fcf * fcf);
  const float f = (float)si * ((float)a.df / (float)N);
  const float q = Af * (f * f) / (fcf + f);
  float sn, cs;
  sincospif(2.0f * q, &sn, &cs);
  return make_float2(fmaf(cs, a.gain, cs) * g, -fmaf(sn, a.gain, sn) * g);
}

// The chirp functions of one call, per channel and row: row c N2 + k2 holds the
// bins i = k2 + N2 k1 of channel c.  The row pass's threads hold bins of
// k1 = j + r N1/R (R the last radix of its forward transform, lgJ = log2(N1/R)),
// and those of even r and of r + 1 lie side by side (chirp_bin), so that one
// 16-byte load gives a lane two of them.  N1 and N are powers of two: shifts,
// not the 64-bit divisions that took most of this kernel's time.
// With a.cov_fill the same launch also sets a.cov_n coverage entries to 1.
__global__ __launch_bounds__(256) void chan_chirp_table_kernel(LargeArgs a, int32_t lgJ,
                                                               float2* __restrict__ hb) {
  const int64_t N = (int64_t)1 << a.lgn;
  const int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (idx < a.cov_n) a.cov_fill[idx] = 1;
  if (idx >= N * a.nchan) return;
  const int c = (int)(idx >> a.lgn);
  const int e = (int)(idx & (N - 1));
  const int64_t i = (e >> a.lg1) + ((int64_t)chirp_bin(e & (a.N1 - 1), lgJ) << a.lg2);
  const double fc = a.f_lo + ((double)c + 0.5) * a.df;
  hb[idx] = chan_chirp(a, fc, i, N);
}

// ---------------------------------------------------------------------------
// rows: forward row DFT, chirp, inverse row DFT, conjugate four-step twiddle
// ---------------------------------------------------------------------------
// Results of a row to its place, times the conjugate twiddle of n1 k2 / N.
template <class SR>
__device__ __forceinline__ void row_store(const float2* v, __amdgpu_buffer_rsrc_t rs, int voff,
                                          const LargeArgs& a, int k2, int tl) {
  constexpr int L = SR::N, R0 = SR::rad_f(0), B0 = L / (R0 * SR::T);
  const uint32_t ph = (uint32_t)k2 << (32 - a.lgn);
#pragma unroll
  for (int b = 0; b < B0; ++b)
#pragma unroll
    for (int r = 0; r < R0; ++r) {
      const int nc = SR::T * b + r * (L / R0);
      const float2 w = expi_phase(ph * (uint32_t)(tl + nc));
      bstore2(rs, cmul(v[b * R0 + r], make_float2(w.x, -w.y)), voff, nc * 8);
    }
}

template <class SR, int G, bool THREE>
__global__ __launch_bounds__(SR::T * G) void rows_kernel(const LargeArgs a) {
  __shared__ float lds[G * (SR::lds_floats() + 1)];
  constexpr int L = SR::N, R0 = SR::rad_f(0), B0 = L / (R0 * SR::T);
  constexpr int RL = SR::rad_f(SR::NP - 1), BL = L / (RL * SR::T);
  const int t = threadIdx.x, g = t / SR::T, tl = t % SR::T;
  const int ngrp = (THREE ? a.un * a.A : a.N2) / G;
  const int64_t item = a.item0 + blockIdx.x / ngrp;
  // (three levels: the rows of a launch's classes, in the order they lie)
  const int row = (THREE ? a.u0 * a.A : 0) + (blockIdx.x % ngrp) * G + g;
  const int lgA = a.lg2 - a.lgB;
  const int k2 = THREE ? (row >> lgA) + ((row & (a.A - 1)) << a.lgB) : row;
  const int c = (int)(item / a.nblocks);
  const int64_t N = (int64_t)a.N1 * a.N2;
  const __amdgpu_buffer_rsrc_t rs = item_rsrc(a.S + (item - a.item0) * N, N * 8);
  const int voff = (row * L + tl) * 8;
  float2 v[SR::E];
#pragma unroll
  for (int b = 0; b < B0; ++b)
#pragma unroll
    for (int r = 0; r < R0; ++r) v[b * R0 + r] = bload2(rs, voff, (SR::T * b + r * (L / R0)) * 8);
  float* my = lds + g * (SR::lds_floats() + 1);
  fft_forward<SR>(v, my, a.twr, tl);
  // chirp on bins i = k2 + N2 k1, from the call's table, two per load
  const __amdgpu_buffer_rsrc_t hs = item_rsrc(a.hb + (int64_t)c * N, N * 8);
  const int hoff = k2 * L * 8 + tl * 16;
#pragma unroll
  for (int b = 0; b < BL; ++b)
#pragma unroll
    for (int r = 0; r < RL; r += 2) {
      const float4 w = __builtin_bit_cast(
          float4, __builtin_amdgcn_raw_buffer_load_b128(
                      hs, hoff, ((r >> 1) * (L / RL) + SR::T * b) * 16, 0));
      v[b * RL + r] = cmul(v[b * RL + r], make_float2(w.x, w.y));
      v[b * RL + r + 1] = cmul(v[b * RL + r + 1], make_float2(w.z, w.w));
    }
  fft_inverse<SR>(v, my, a.twr, tl);
  row_store<SR>(v, rs, voff, a, k2, tl);
}

// ---------------------------------------------------------------------------
// cols_inv: inverse column DFT, overlap-save window, detection, voltages
// ---------------------------------------------------------------------------
// Three-level form (THREE): for each a, the inverse DFTs over kb of rows
// a + A kb give the samples n2 = a + A b.
template <class SC, int G, bool THREE>
__global__ __launch_bounds__(SC::T * G) void cols_inv_kernel(const LargeArgs a) {
  // run pitch of the detected samples in LDS; columns above 512 points have no
  // room for the pad beside a second workgroup
  constexpr int QP = SC::N <= 512 ? G + 4 : G;
  constexpr int LDSF = G * (SC::lds_floats() + 1);
  __shared__ __align__(16) float lds[LDSF > QP * SC::N ? LDSF : QP * SC::N];
  constexpr int L = SC::N, RI = SC::rad_i(0), BI = L / (RI * SC::T);
  constexpr int R0 = SC::rad_f(0), B0 = L / (R0 * SC::T);
  const int t = threadIdx.x, g = t % G, tl = t / G;
  const int ngrp = a.N1 / G;
  const int nsub = THREE ? a.A : 1;
  const int64_t item = a.item0 + blockIdx.x / ((unsigned)ngrp * nsub);
  const int rem = (int)(blockIdx.x % ((unsigned)ngrp * nsub));
  const int sa = THREE ? rem / ngrp : 0;  // a of this column run
  const int sA = THREE ? a.A : 1;         // n2 = sa + sA * (local index)
  const int n1 = (rem % ngrp) * G + g;
  const int c = (int)(item / a.nblocks);
  const int64_t k = item - (int64_t)c * a.nblocks;
  const int64_t N = (int64_t)a.N1 * a.N2;
  const __amdgpu_buffer_rsrc_t rs = item_rsrc(a.S + (item - a.item0) * N, N * 8);
  const int pitch = a.N1 * sA;  // columns between successive local indices
  const int v0 = n1 + a.N1 * sa + tl * pitch;
  float2 v[SC::E];
#pragma unroll
  for (int b = 0; b < BI; ++b)
#pragma unroll
    for (int r = 0; r < RI; ++r)
      v[b * RI + r] = bload2(rs, v0 * 8, (SC::T * b + r * (L / RI)) * pitch * 8);
  fft_inverse<SC>(v, lds + g * (SC::lds_floats() + 1), a.twc, tl);
  // sample m = n - nfront of the block's window is kept if 0 <= m < lim; with
  // the voltages' resource ending at lim, stores outside the window fall away
  // (a negative m is past the end as an unsigned offset)
  const int64_t left = a.nsamp - k * a.M;
  const int lim = (int)(left < a.M ? left : a.M);
  const int m0 = v0 - a.nfront;
  const int64_t o0 = (int64_t)c * a.nsamp + k * a.M;
  if (a.vout) {
    const __amdgpu_buffer_rsrc_t vs = item_rsrc(a.vout + o0, (int64_t)lim * 8);
#pragma unroll
    for (int b = 0; b < B0; ++b)
#pragma unroll
      for (int r = 0; r < R0; ++r)
        bstore2(vs, v[b * R0 + r], (m0 + (SC::T * b + r * (L / R0)) * pitch) * 8, 0);
  }
  if (!a.fuse) {
#pragma unroll
    for (int b = 0; b < B0; ++b)
#pragma unroll
      for (int r = 0; r < R0; ++r) {
        const int m = m0 + (SC::T * b + r * (L / R0)) * pitch;
        const float2 z = v[b * R0 + r];
        if ((unsigned)m < (unsigned)lim) a.p[o0 + m] = z.x * z.x + z.y * z.y;
      }
    return;
  }
  // Fused detection and integration.  The workgroup holds, for each of its
  // n2, the run of G consecutive samples n = n1b + N1 n2 + g (g < G).  |z|^2
  // of the kept samples goes to LDS as [local n2][g], QP words a run (a pad of
  // four words spreads the runs over the banks and keeps them 16-byte
  // aligned); groups of n_int start where n = nfront (mod n_int).  Groups
  // inside a run are summed here and stored; a group split across the end of
  // one run and the start of the next is left as two partial sums for
  // integrate_fixup_kernel.
  __syncthreads();  // the transform's last LDS reads are done
  float* q = lds;
#pragma unroll
  for (int b = 0; b < B0; ++b)
#pragma unroll
    for (int r = 0; r < R0; ++r) {
      const int nc = SC::T * b + r * (L / R0);
      const float2 z = v[b * R0 + r];
      const bool kept = (unsigned)(m0 + nc * pitch) < (unsigned)lim;
      q[(tl + nc) * QP + g] = kept ? z.x * z.x + z.y * z.y : 0.f;
    }
  __syncthreads();
  const int ni = a.n_int;                          // a power of two, at most G
  const int phi = a.nfront & (ni - 1);
  const int per_run = G / ni;                      // group starts per run
  const int lgr = 31 - __builtin_clz(per_run);
  const int n1b = n1 - g;
  const int64_t item_local = item - a.item0;
  float* part = a.p + item_local * (N / G) * 2;
  float* Pu = a.P + (int64_t)c * a.t_int + k * a.M / ni;  // n_int divides M
  const int64_t ul = a.t_int - k * a.M / ni;
  const int ulim = (int)(ul < a.M / ni ? ul : a.M / ni);
  for (int j = threadIdx.x; j < (L << lgr); j += SC::T * G) {
    const int nl = j >> lgr, slot = j & (per_run - 1);
    const float* run = q + nl * QP;
    const int n0 = n1b + a.N1 * (sa + sA * nl);    // run's first sample
    const int s0 = phi + slot * ni;                // group start within the run
    if (s0 + ni > G) {
      // the split group: partial sums of the head [0, phi) and the tail [G - ni + phi, G)
      float h = 0.f, t = 0.f;
      for (int i = 0; i < phi; ++i) h += run[i];
      for (int i = G - ni + phi; i < G; ++i) t += run[i];
      part[2 * (n0 / G)] = h;
      part[2 * (n0 / G) + 1] = t;
      continue;
    }
    const int m = n0 + s0 - a.nfront;              // a multiple of n_int
    if (m < 0) continue;
    const int u = m / ni;
    if (u >= ulim) continue;
    float acc = 0.f;
    if ((ni & 3) == 0 && (phi & 3) == 0) {
      for (int i = 0; i < ni; i += 4) {
        const float4 x = *(const float4*)(run + s0 + i);
        acc += x.x;
        acc += x.y;
        acc += x.z;
        acc += x.w;
      }
    } else {
      for (int i = 0; i < ni; ++i) acc += run[s0 + i];
    }
    Pu[u] = acc;
  }
}

// The integration groups split across two runs of G samples: the tail of
// run j plus the head of run j + 1 (partial sums from cols_inv_kernel).
__global__ __launch_bounds__(256) void integrate_fixup_kernel(const LargeArgs a, int32_t G,
                                                              int64_t items) {
  const int64_t runs = (int64_t)a.N1 * a.N2 / G;
  const int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (idx >= items * (runs - 1)) return;
  const int64_t item_local = idx / (runs - 1);
  const int64_t j = idx - item_local * (runs - 1);
  const int64_t item = a.item0 + item_local;
  const int c = (int)(item / a.nblocks);
  const int64_t k = item - (int64_t)c * a.nblocks;
  const int ni = a.n_int;
  const int phi = (int)(a.nfront % ni);
  const int64_t start = j * G + G - ni + phi;  // first sample of the split group
  const int64_t m = start - a.nfront;
  if (m < 0 || m >= a.M) return;
  const int64_t u = (k * a.M + m) / ni;
  if (u >= a.t_int) return;
  const float* part = a.p + item_local * runs * 2;
  a.P[(int64_t)c * a.t_int + u] = part[2 * j + 1] + part[2 * (j + 1)];
}

// P[c][u] = sum_{r < n_int} p[c][u n_int + r] in ascending r, grid (u
// blocks, channels).  V consecutive samples per load (V divides n_int and
// the channel stride, so every vector load is aligned).
template <int V>
__global__ __launch_bounds__(256) void integrate_kernel(const float* __restrict__ p,
                                                        float* __restrict__ P, int64_t nsamp,
                                                        int64_t t_int, int32_t n_int) {
  using VT = typename std::conditional<V == 4, float4, typename std::conditional<
                                                         V == 2, float2, float>::type>::type;
  const int c = blockIdx.y;
  const int64_t u = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (u >= t_int) return;
  const VT* pc = (const VT*)(p + (int64_t)c * nsamp + u * n_int);
  float s = 0.f;
  for (int r = 0; r < n_int / V; ++r) {
    const VT x = pc[r];
    if constexpr (V == 4) {
      s += x.x;
      s += x.y;
      s += x.z;
      s += x.w;
    } else if constexpr (V == 2) {
      s += x.x;
      s += x.y;
    } else {
      s += x;
    }
  }
  P[(int64_t)c * t_int + u] = s;
}

static int launch_integrate(const float* p, float* P, int64_t nsamp, int64_t t_int,
                            int32_t n_int, int32_t nchan, hipStream_t st) {
  const int64_t nb = (t_int + 255) / 256;
  if (nb > 0x7fffffffLL || nchan > 65535) return (int)hipErrorInvalidValue;
  if (nb == 0) return 0;
  const dim3 grid((unsigned)nb, (unsigned)nchan);
  if (n_int % 4 == 0 && (nchan == 1 || nsamp % 4 == 0))
    hipLaunchKernelGGL(integrate_kernel<4>, grid, dim3(256), 0, st, p, P, nsamp, t_int, n_int);
  else if (n_int % 2 == 0 && (nchan == 1 || nsamp % 2 == 0))
    hipLaunchKernelGGL(integrate_kernel<2>, grid, dim3(256), 0, st, p, P, nsamp, t_int, n_int);
  else
    hipLaunchKernelGGL(integrate_kernel<1>, grid, dim3(256), 0, st, p, P, nsamp, t_int, n_int);
  return (int)hipGetLastError();
}

// The split integration groups of one chunk of items (fused path); none when
// the groups start on run boundaries.
static int launch_fixup(const LargeArgs& a, int G, int64_t items, hipStream_t st) {
  if (a.nfront % a.n_int == 0) return 0;
  const int64_t runs = (int64_t)a.N1 * a.N2 / G;
  const int64_t n = items * (runs - 1);
  const int64_t nb = (n + 255) / 256;
  if (nb > 0x7fffffffLL) return (int)hipErrorInvalidValue;
  if (nb == 0) return 0;
  hipLaunchKernelGGL(integrate_fixup_kernel, dim3((unsigned)nb), dim3(256), 0, st, a, G, items);
  return (int)hipGetLastError();
}

// ---------------------------------------------------------------------------
// Full-band mode: one real series over the whole band (Sec. 2.1, 2.3, 3.1)
// ---------------------------------------------------------------------------
// A real block of 2N samples is transformed as N complex points z[n] =
// x[2n] + i x[2n+1].  With Z = DFT_N(z), the spectra of the even and odd
// samples are E_i = (Z_i + conj Z_(N-i)) / 2 and O_i = (Z_i - conj Z_(N-i)) /
// (2i), and the real spectrum is X_i = E_i + w^i O_i, X_(N-i) = conj(E_i -
// w^i O_i), w = exp(-i pi / N).  After the filter, Y = H X, the same relations
// taken backwards give Z', whose inverse DFT holds the filtered samples in
// pairs.  In the four-step layout bin i = k2 + N2 k1 sits in row k2 and its
// mirror N - i in row N2 - k2 at k1' = N1 - 1 - k1 (row 0: k1' = -k1 mod N1),
// so one workgroup transforms rows k2 and N2 - k2 together and hands each
// row to the other through LDS.
__device__ __forceinline__ float2 tw2_fwd(const LargeArgs& a, uint32_t m) {
  return expi_phase(m << (31 - a.lgn));  // m / 2N turns
}

// Chirp of Eq. 3 about the lower band edge at real-spectrum bin j (0 .. N):
// f = j bw / N above f_lo, q = D DM f^2 / (f_lo^2 (f_lo + f)) = qb j^2 /
// (1 + qbeta j) turns in FP64, reduced before the FP32 rotation; times the
// band taper at x = j/N - 1/2 and the 1/N of the inverse transform.  The
// quotient (1 + qbeta j lies in [1, 3)) takes the hardware's reciprocal, two
// Newton steps and one correction of the quotient itself.
__device__ __forceinline__ float2 band_chirp(const LargeArgs& a, uint32_t j, float inv_n) {
  const double s = (double)j;
  const double num = a.qb * (s * s), den = fma(a.qbeta, s, 1.0);
  double r = __builtin_amdgcn_rcp(den);
  r = fma(r, fma(-den, r, 1.0), r);
  r = fma(r, fma(-den, r, 1.0), r);
  double q = num * r;
  q = fma(r, fma(-den, q, num), q);
  const float2 h = expi_neg_turns_fp32(q - rint(q), RotationSize{1.0f, a.gain});
  const float g = inv_n * taper_gain<false>(a.taper, (float)j * inv_n - 0.5f);
  return make_float2(h.x * g, h.y * g);
}

// The chirp function of one call for every real-spectrum bin, shared by all
// blocks of the record, in the order the row pass reads it: entry
// k2 N1 + k1 holds bin j = k2 + N2 k1 (j < N), entry N the Nyquist bin.  Two
// neighbouring entries per store, IT of those per thread.  (N1 is a power of
// two: shifts, not 64-bit divisions.)
template <int IT>
__global__ __launch_bounds__(256) void band_chirp_table_kernel(LargeArgs a,
                                                               float2* __restrict__ hb) {
  const uint32_t N = 1u << a.lgn;
  const float inv_n = 1.0f / (float)N;
  for (int i = 0; i < IT; ++i) {
    const uint32_t e = ((blockIdx.x * IT + i) * 256 + threadIdx.x) * 2;
    if (e >= N) break;
    const uint32_t j = (e >> a.lg1) + ((e & (uint32_t)(a.N1 - 1)) << a.lg2);
    const float2 p = band_chirp(a, j, inv_n), q = band_chirp(a, j + (uint32_t)a.N2, inv_n);
    *(float4*)(hb + e) = make_float4(p.x, p.y, q.x, q.y);
  }
  if (blockIdx.x == 0 && threadIdx.x == 0) hb[N] = band_chirp(a, N, inv_n);
}

template <int L, int LDSF>
constexpr int pair_stride() {
  return 2 * L > LDSF + 1 ? 2 * L : ((LDSF + 1 + 3) & ~3);
}

// One mirror pair of the packed spectrum: from Z_i and Z_(N-i) (z, zm) to
// the filtered Z'_i and Z'_(N-i).  With E' = (Y_i + conj Y_(N-i)) / 2 and
// O' = (Y_i - conj Y_(N-i)) conj(w^i) / 2, Z'_i = E' + i O' and
// Z'_(N-i) = conj(E') + i conj(O').
__device__ __forceinline__ void real_pair(const LargeArgs& a, uint32_t i, float2 hp, float2 hm,
                                          float2 z, float2 zm, float2* zi, float2* zmi) {
  const float2 e = make_float2(0.5f * (z.x + zm.x), 0.5f * (z.y - zm.y));
  const float2 o = make_float2(0.5f * (z.y + zm.y), -0.5f * (z.x - zm.x));
  const float2 w = tw2_fwd(a, i);
  const float2 wo = cmul(w, o);
  float2 yp = cmul(cadd(e, wo), hp);
  float2 ym = cmul(make_float2(e.x - wo.x, wo.y - e.y), hm);
  if (i == 0) {  // DC and Nyquist of a real series are real
    yp.y = 0.f;
    ym.y = 0.f;
  }
  const float2 e2 = make_float2(0.5f * (yp.x + ym.x), 0.5f * (yp.y - ym.y));
  const float2 o2 = cmul(make_float2(0.5f * (yp.x - ym.x), 0.5f * (yp.y + ym.y)),
                         make_float2(w.x, -w.y));
  *zi = make_float2(e2.x - o2.y, e2.y + o2.x);
  *zmi = make_float2(e2.x + o2.y, o2.x - e2.y);
}

// FLY: the chirp is formed here instead of being read from the call's table.
template <class SR, int G, bool FLY, bool THREE>
__global__ __launch_bounds__(SR::T * G) void rows_real_kernel(const LargeArgs a) {
  constexpr int L = SR::N, STRIDE = pair_stride<SR::N, SR::lds_floats()>();
  __shared__ __align__(16) float lds[G * STRIDE];
  constexpr int R0 = SR::rad_f(0), B0 = L / (R0 * SR::T);
  constexpr int RL = SR::rad_f(SR::NP - 1), BL = L / (RL * SR::T);
  const int t = threadIdx.x, g = t / SR::T, tl = t % SR::T;
  // N2/2 row pairs per item, G/2 per workgroup: (0, N2/2), then (k, N2 - k);
  // with three levels A pairs per pair of mirror classes
  const int ngrp = (THREE ? 2 * a.un * a.A : a.N2) / G;
  const int64_t item = a.item0 + blockIdx.x / ngrp;
  int pair = (blockIdx.x % ngrp) * (G / 2) + (g >> 1);
  if constexpr (THREE) {
    const int lgA = a.lg2 - a.lgB;
    const int u = a.u0 + (pair >> lgA), ka = pair & (a.A - 1), B = 1 << a.lgB;
    pair = u ? u + B * ka : ka < a.A / 2 ? B * ka : B / 2 + B * (ka - a.A / 2);
  }
  const int side = g & 1;
  const int k2 = pair == 0 ? side * (a.N2 / 2) : (side ? a.N2 - pair : pair);
  const int64_t N = (int64_t)a.N1 * a.N2;
  const __amdgpu_buffer_rsrc_t rs = item_rsrc(a.S + (item - a.item0) * N, N * 8);
  const int voff = ((int)spec_row(a, k2) * L + tl) * 8;
  float2 v[SR::E];
#pragma unroll
  for (int b = 0; b < B0; ++b)
#pragma unroll
    for (int r = 0; r < R0; ++r) v[b * R0 + r] = bload2(rs, voff, (SR::T * b + r * (L / R0)) * 8);
  float* my = lds + g * STRIDE;
  fft_forward<SR>(v, my, a.twr, tl);
  __syncthreads();  // every read of the last exchange is done
  float2* mine = (float2*)my;
#pragma unroll
  for (int b = 0; b < BL; ++b)
#pragma unroll
    for (int r = 0; r < RL; ++r) mine[tl + SR::T * b + r * (L / RL)] = v[b * RL + r];
  __syncthreads();
  // Each mirror pair is filtered once, in place.  A row pair (k, N2 - k):
  // bin k1 of row k pairs with N1 - 1 - k1 of row N2 - k; side s takes
  // k1 in [s N1/2, (s+1) N1/2).  Row 0 pairs k1 with -k1 mod N1 (k1 = 0 and
  // N1/2 with themselves); row N2/2 pairs k1 with N1 - 1 - k1.
  float2* rowA = (float2*)(lds + (pair == 0 ? g : (g & ~1)) * STRIDE);
  float2* rowB = (float2*)(lds + (pair == 0 ? g : (g | 1)) * STRIDE);
  const int kA = pair == 0 ? k2 : pair;
  const int kB = pair == 0 ? k2 : a.N2 - pair;
  const float2* hA = a.hb + (int64_t)kA * L;  // chirp of row kA's bins, then row kB's
  const float2* hB = a.hb + (int64_t)kB * L;
  const float inv_n = 1.0f / (float)N;
  auto chirp = [&](const float2* h, int row, int k1) {
    if constexpr (FLY) {
      (void)h;
      return band_chirp(a, (uint32_t)row + ((uint32_t)k1 << a.lg2), inv_n);
    } else {
      return h[k1];
    }
  };
  constexpr int half = L / 2;
  if (pair != 0) {
    // two neighbouring bins and their mirrors per step: 16-byte accesses
#pragma unroll 2
    for (int p = 2 * tl; p < half; p += 2 * SR::T) {
      const int k1 = p + side * half, k1m = L - 2 - k1;  // bins k1, k1 + 1; k1m + 1, k1m
      float4 h4, m4;
      if constexpr (FLY) {
        const float2 p0 = chirp(hA, kA, k1), p1 = chirp(hA, kA, k1 + 1);
        const float2 q0 = chirp(hB, kB, k1m), q1 = chirp(hB, kB, k1m + 1);
        h4 = make_float4(p0.x, p0.y, p1.x, p1.y);
        m4 = make_float4(q0.x, q0.y, q1.x, q1.y);
      } else {
        h4 = *(const float4*)(hA + k1);
        m4 = *(const float4*)(hB + k1m);
      }
      const float4 z4 = *(const float4*)(rowA + k1), y4 = *(const float4*)(rowB + k1m);
      float2 za, zb, ya, yb;
      real_pair(a, (uint32_t)kA + ((uint32_t)k1 << a.lg2), make_float2(h4.x, h4.y),
                make_float2(m4.z, m4.w), make_float2(z4.x, z4.y), make_float2(y4.z, y4.w), &za,
                &yb);
      real_pair(a, (uint32_t)kA + ((uint32_t)(k1 + 1) << a.lg2), make_float2(h4.z, h4.w),
                make_float2(m4.x, m4.y), make_float2(z4.z, z4.w), make_float2(y4.x, y4.y), &zb,
                &ya);
      *(float4*)(rowA + k1) = make_float4(za.x, za.y, zb.x, zb.y);
      *(float4*)(rowB + k1m) = make_float4(ya.x, ya.y, yb.x, yb.y);
    }
  } else {
    for (int p = tl; p < half; p += SR::T) {
      const int k1 = p, k1m = side == 0 ? (L - p) & (L - 1) : L - 1 - p;
      float2 zi, zmi;
      const uint32_t i = (uint32_t)kA + ((uint32_t)k1 << a.lg2);
      // (the mirror of bin 0 is the Nyquist bin, N = row 0 at k1 = N1)
      const float2 hm = i == 0 ? chirp(a.hb + N - L, 0, L) : chirp(hB, kB, k1m);
      real_pair(a, i, chirp(hA, kA, k1), hm, rowA[k1], rowB[k1m], &zi, &zmi);
      rowA[k1] = zi;
      rowB[k1m] = zmi;
      if (side == 0 && p == 0) {
        const float2 hh = chirp(hA, kA, half);
        real_pair(a, (uint32_t)half << a.lg2, hh, hh, rowA[half], rowA[half], &zi, &zmi);
        rowA[half] = zi;
      }
    }
  }
  __syncthreads();
#pragma unroll
  for (int b = 0; b < BL; ++b)
#pragma unroll
    for (int r = 0; r < RL; ++r) v[b * RL + r] = mine[tl + SR::T * b + r * (L / RL)];
  fft_inverse<SR>(v, my, a.twr, tl);  // its first exchange waits for the reads above
  row_store<SR>(v, rs, voff, a, k2, tl);
}

// Inverse transform of recorded spectra (Sec. 2.3, 3.1).  Record s holds
// bins 0 .. L-1 of a 2L-point real FFT as int8 (re, im); the Nyquist bin is
// not recorded and the DC bin's imaginary part is dropped.  Packed as above
// (with w = exp(-i pi / L) and X_L = 0), the record becomes L complex values
// Z_c = (E_c + i O_c), whose inverse DFT (times 1/L) is the record's 2L real
// samples in pairs.  A group of SC::T lanes handles one record; G records
// per workgroup.  The workgroups loop over groups of G records (grid-stride),
// each lane holding the next group's words in registers while the current
// group is transformed and stored, so loads, transforms and stores of
// different groups overlap instead of every workgroup loading, then
// transforming, then storing at the same time.
template <class SC, int G>
__global__ __launch_bounds__(SC::T * G) void gsb_inverse_kernel(
    const uint32_t* __restrict__ spec, float2* __restrict__ out,
    const float2* __restrict__ pre, const float2* __restrict__ tw, int64_t nspec) {
  constexpr int L = SC::N, STRIDE = pair_stride<SC::N, SC::lds_floats()>();
  constexpr int W = L / 2 / SC::T;  // words (two bins each) per lane per record
  static_assert(STRIDE % 4 == 0, "records are staged as float4");
  static_assert(W * SC::T == L / 2, "lanes tile a record's words");
  __shared__ __align__(16) float lds[G * STRIDE];
  constexpr int RI = SC::rad_i(0), BI = L / (RI * SC::T);
  constexpr int R0 = SC::rad_f(0), B0 = L / (R0 * SC::T);
  const int t = threadIdx.x, g = t / SC::T, tl = t % SC::T;
  const int64_t ngroups = (nspec + G - 1) / G;
  float* my = lds + g * STRIDE;
  float4* X4 = (float4*)my;
  const float sc = 0.5f / (float)L;
  uint32_t wd[W];
  auto fetch = [&](int64_t grp) {
    const int64_t s = grp * G + g;
    const bool ok = grp < ngroups && s < nspec;
#pragma unroll
    for (int j = 0; j < W; ++j) wd[j] = ok ? spec[s * (L / 2) + tl + SC::T * j] : 0u;
  };
  fetch(blockIdx.x);
  for (int64_t grp = blockIdx.x; grp < ngroups; grp += gridDim.x) {
    const int64_t s = grp * G + g;
    const bool live = s < nspec;
    __syncthreads();  // the previous group's transform is done with the LDS
#pragma unroll
    for (int j = 0; j < W; ++j) {
      const uint32_t w = wd[j];
      X4[tl + SC::T * j] = make_float4((float)(int8_t)(w & 0xffu),
                                       (float)(int8_t)((w >> 8) & 0xffu),
                                       (float)(int8_t)((w >> 16) & 0xffu),
                                       (float)(int8_t)(w >> 24));
    }
    fetch(grp + gridDim.x);  // in flight during this group's transform
    __syncthreads();
    const float2* X = (const float2*)my;
    float2 v[SC::E];
#pragma unroll
    for (int b = 0; b < BI; ++b)
#pragma unroll
      for (int r = 0; r < RI; ++r) {
        const int c = tl + SC::T * b + r * (L / RI);
        float2 x = X[c];
        float2 m = make_float2(0.f, 0.f);
        if (c == 0)
          x.y = 0.f;
        else
          m = X[L - c];
        const float2 e = make_float2(x.x + m.x, x.y - m.y);                    // 2 E_c
        const float2 o = cmul(make_float2(x.x - m.x, x.y + m.y), pre[c]);      // 2 O_c
        v[b * RI + r] = make_float2(sc * (e.x - o.y), sc * (e.y + o.x));
      }
    fft_inverse<SC>(v, my, tw, tl);  // its first exchange waits for the reads above
    if (live) {
#pragma unroll
      for (int b = 0; b < B0; ++b)
#pragma unroll
        for (int r = 0; r < R0; ++r) out[s * L + tl + SC::T * b + r * (L / R0)] = v[b * R0 + r];
    }
  }
}

// ---------------------------------------------------------------------------
// Host side
// ---------------------------------------------------------------------------
constexpr int64_t kChunkBytes = (int64_t)512 << 20;  // intermediate spectra per chunk

bool large_supported(int N) { return N >= (1 << 15) && N <= (1 << 26) && (N & (N - 1)) == 0; }

// The fused integration leaves two partial sums per run of G >= 8 samples
// of every item of a chunk in the |y|^2 buffer: at most N bytes per item.
size_t large_partial_bytes(int64_t N, int64_t items) { return (size_t)items * (size_t)N; }

int64_t large_chunk_items(const BeamPlan& p) {
  const int64_t items = (int64_t)p.nchan * p.nblocks;
  const int64_t per = std::max<int64_t>(1, kChunkBytes / ((int64_t)p.N * 8));
  return std::min(items, per);
}

// How an N = 2^LGN point transform is split: N1 = 2^LG1 (rows), and the
// column dimension N2 = A B with A = 2^LGA, B = 2^LGB.  Up to 2^22 points
// two levels; beyond, three, with every sub-transform between 128 and 2048
// points.  Up to 2^22 the columns are 2^(LGN/2) long, except from 2^16 to
// 2^20 points, where columns half as long (rows twice as long) measured
// faster: the column passes then hold half the data per workgroup and more
// workgroups fit on a CU (2^18-point channel transforms 0.175 -> 0.168 ms per
// call on the 2^23-sample single-channel workload; the full band at 2^19,
// 2^20 and 2^21 real points 0.195 -> 0.184, 0.162 -> 0.144 and 0.181 ->
// 0.153 ms, with the row groups below).
template <int LGN>
struct Split {
  static constexpr int LGA = LGN <= 22 ? 0 : (LGN >= 26 ? 8 : 7);
  static constexpr int LGB = LGN > 22 ? 7 : (LGN >= 16 && LGN <= 20) ? LGN / 2 - 1 : LGN / 2;
  static constexpr int LG1 = LGN - LGA - LGB;
  static constexpr int N1 = 1 << LG1, A = 1 << LGA, B = 1 << LGB, N2 = A * B;
  static constexpr bool THREE = LGA > 0;
  using SC = typename SubSched<B>::type;                   // last column sub-transform
  using SA = typename SubSched<THREE ? A : 128>::type;     // middle one (three levels)
  using SR = typename SubSched<N1>::type;                  // rows
  static constexpr int GC = SC::T * 16 <= 1024 ? 16 : 8;
  // The forward column pass of the two-level channel transforms takes 32
  // adjacent columns per workgroup where that stays within 512 threads
  // (columns of up to 256 points): 256-byte runs instead of 128.  Measured
  // on the single-channel workload (2^18 = 1024 x 256): 0.158 -> 0.154 ms
  // per call at 2^23 samples, 1.31 -> 1.28 ms at 2^26.  The inverse pass
  // (0.153 -> 0.158 ms that way) and the full band's forward pass (2048-point
  // rows, 16 KB between the rows of a run) keep GC.
  static constexpr int GW = !THREE && SC::T * GC * 2 <= 512 ? 2 * GC : GC;
  static constexpr int GA = SA::T * 16 <= 1024 ? 16 : 8;
  static_assert(LG1 >= 7 && LG1 <= 11 && N1 % GC == 0 && N1 % GW == 0 && N1 % GA == 0,
                "sub-transforms of 128 .. 2048 points, column groups tiling N1");
};

// Rows per workgroup of the row pass (T threads per row): at most eight and
// at most 256 threads.  Small workgroups let several be resident per CU at
// different phases (loads of one beside the transforms of another); 1024-point
// rows four to a workgroup instead of eight: 0.168 -> 0.158 ms per call on
// the 2^23-sample single-channel workload; 2048-point rows two instead of
// four: 2^22-point channel transforms 1.40 -> 1.37 ms, full band at 2^20
// real points 0.156 -> 0.144 ms.  (With the real series each workgroup holds
// mirror-row pairs, so the count stays even.)
constexpr int rows_per_group(int T) { return T * 8 <= 256 ? 8 : 256 / T; }

// Relative gain correction of a whole transform pair (see gain_correction): its
// sub-transforms, and one hardware rotation each way per level above the first.
template <int LGN>
static float split_gain() {
  using SP = Split<LGN>;
  double g = gain_of<typename SP::SC>() + gain_of<typename SP::SR>();
  if (SP::THREE) g += gain_of<typename SP::SA>();
  return (float)(g - 2.0 * (SP::THREE ? 2 : 1) * kHwRotationGain);
}

// Fill the split-dependent fields of a and its sub-transform twiddles.
template <int LGN>
static int set_split(LargeArgs& a) {
  using SP = Split<LGN>;
  int e = twiddles_of<typename SP::SC>(&a.twc);
  if (!e) e = twiddles_of<typename SP::SR>(&a.twr);
  if (!e && SP::THREE) e = twiddles_of<typename SP::SA>(&a.twm);
  a.N1 = SP::N1;
  a.N2 = SP::N2;
  a.A = SP::A;
  a.lgB = SP::LGB;
  a.lg2 = SP::LGA + SP::LGB;
  a.lgn = LGN;
  a.lg1 = SP::LG1;
  a.gain = split_gain<LGN>();
  return e;
}

// The spectra that a run of passes works through stay in the 256 MiB memory-side
// cache: between HBM-bound passes (4.9 TB/s copied) of 512 MiB each nothing was
// left of them there.  A launch of passes takes the items, and the middle and row
// passes of longer transforms the column classes, that fit: 192 MiB where the
// call's chirp table is read beside them, 256 MiB without one.  Measured per call,
// against 512 MiB: one channel of 2^25 samples at 2^18 points 525 -> 460 us, at
// 2^23 points 727 -> 615 us; full band of 2^27 samples at 2^19 points 1.27 -> 1.12
// ms, at 2^26 points 2.40 -> 2.10 ms, at 2^27 points 2.31 -> 2.15 ms.  (64 and
// 128 MiB: 539 and 477, 643 and 610 us; 1.38 and 1.16, 2.11 and 2.12, 2.40 and
// 2.23 ms: small launches end in a nearly empty round of workgroups.)
constexpr int64_t kCacheBytes = (int64_t)256 << 20;
static int64_t cached_bytes(const LargeArgs& a) {
  return a.hb ? kCacheBytes / 4 * 3 : kCacheBytes;
}
// Launches of each pass for one call of `items` items, at most a chunk each.
static int64_t cached_launches(const LargeArgs& a, int64_t items, int64_t chunk) {
  const int64_t most = std::max<int64_t>(1, cached_bytes(a) / ((int64_t)a.N1 * a.N2 * 8));
  const int64_t n = std::min(most, chunk);
  return (items + n - 1) / n;
}

// The passes over one chunk of q items (blocks of one or more channels):
// columns forward, rows (chirp; REAL: the mirror-pair filter of the real
// series), columns inverse with the kept window, detection and (fused)
// integration.  GR rows per workgroup.  After the first half of a three-level
// column transform the rows of one class kb (with the mirror pairs of the real
// series: of kb and B - kb) need no others until the last pass, so the passes in
// between take as many classes at a time as stay in the cache.
template <int LGN, int DT, bool REAL, int GR>
static int run_passes(const LargeArgs& a, int64_t q, hipStream_t st) {
  using SP = Split<LGN>;
  using SC = typename SP::SC;
  using SA = typename SP::SA;
  using SR = typename SP::SR;
  constexpr int GC = SP::GC, GA = SP::GA;
  static_assert(SP::N2 % GR == 0 && (!REAL || GR % 2 == 0) && (!SP::THREE || SP::A % GR == 0),
                "row groups tile N2 and its classes");
  constexpr int GF = REAL ? GC : SP::GW;
  constexpr bool TH = SP::THREE;
  constexpr int NU = !TH ? 1 : REAL ? SP::B / 2 : SP::B;  // classes (or pairs of them)
  const int64_t gc = q * SP::A * (SP::N1 / GC), gf = q * SP::A * (SP::N1 / GF);
  const int64_t ga = q * SP::B * (SP::N1 / GA), gr = q * (SP::N2 / GR);
  if (gc > 0x7fffffffLL || gf > 0x7fffffffLL || ga > 0x7fffffffLL || gr > 0x7fffffffLL)
    return (int)hipErrorInvalidValue;
  hipLaunchKernelGGL((cols_fwd_kernel<SC, GF, DT, TH>), dim3((unsigned)gf), dim3(SC::T * GF), 0,
                     st, a);
  const int64_t unit_bytes = q * ((int64_t)SP::N1 * SP::N2 * 8 / NU);
  const int per = TH ? (int)std::max<int64_t>(1, std::min<int64_t>(NU, cached_bytes(a) / unit_bytes)) : 1;
  LargeArgs b = a;
  for (b.u0 = 0; b.u0 < NU; b.u0 += per) {
    b.un = std::min(per, NU - b.u0);
    const unsigned na = (unsigned)(ga / NU * b.un), nr = (unsigned)(gr / NU * b.un);
    if constexpr (TH)
      hipLaunchKernelGGL((cols_mid_kernel<SA, GA, false, REAL>), dim3(na), dim3(SA::T * GA), 0, st,
                         b);
    if constexpr (REAL) {
      if (a.hb)
        hipLaunchKernelGGL((rows_real_kernel<SR, GR, false, TH>), dim3(nr), dim3(SR::T * GR), 0,
                           st, b);
      else
        hipLaunchKernelGGL((rows_real_kernel<SR, GR, true, TH>), dim3(nr), dim3(SR::T * GR), 0, st,
                           b);
    } else {
      hipLaunchKernelGGL((rows_kernel<SR, GR, TH>), dim3(nr), dim3(SR::T * GR), 0, st, b);
    }
    if constexpr (TH)
      hipLaunchKernelGGL((cols_mid_kernel<SA, GA, true, REAL>), dim3(na), dim3(SA::T * GA), 0, st,
                         b);
  }
  hipLaunchKernelGGL((cols_inv_kernel<SC, GC, SP::THREE>), dim3((unsigned)gc), dim3(SC::T * GC),
                     0, st, a);
  int e = 0;
  if (a.fuse && (e = launch_fixup(a, GC, q, st))) return e;
  return (int)hipGetLastError();
}

template <int LGN>
static int launch_large_t(const BeamPlan& p, const void* xt, double dm, float2* S, float* pbuf,
                          float* P, void* vout, int exact_div, int32_t* cov_fill, int64_t cov_n,
                          void* stream) {
  using SP = Split<LGN>;
  using SR = typename SP::SR;
  constexpr int GR = rows_per_group(SR::T);
  LargeArgs a{};
  int e = set_split<LGN>(a);
  if (e) return e;
  a.x = xt;
  a.S = S;
  a.p = pbuf;
  a.vout = (float2*)vout;
  a.nsamp = p.nsamp;
  a.nblocks = p.nblocks;
  a.nchan = p.nchan;
  a.M = p.M;
  a.nfront = p.nfront;
  a.phase_mode = p.phase_mode;
  a.taper = p.taper;
  a.exact_div = exact_div;
  a.f_lo = p.f_lo;
  a.df = p.df;
  a.dconst = p.dconst;
  a.dm = dm;
  a.P = P;
  a.t_int = p.t_int;
  a.n_int = p.n_int;
  a.fuse = SP::GC % p.n_int == 0 ? 1 : 0;
  a.cov_fill = cov_fill;
  a.cov_n = cov_fill ? cov_n : 0;
  hipStream_t st = (hipStream_t)stream;
  const int64_t items = (int64_t)p.nchan * p.nblocks;
  const int64_t chunk = large_chunk_items(p);
  // the call's chirp table follows the chunk of spectra in the workspace
  constexpr int64_t NP = (int64_t)1 << LGN;
  a.hb = S + chunk * NP;
  const int64_t nt = (std::max<int64_t>(NP * p.nchan, a.cov_n) + 255) / 256;
  if (nt > 0x7fffffffLL) return (int)hipErrorInvalidValue;
  constexpr int LGJ = SP::LG1 - (31 - __builtin_clz(SR::rad_f(SR::NP - 1)));
  hipLaunchKernelGGL(chan_chirp_table_kernel, dim3((unsigned)nt), dim3(256), 0, st, a, LGJ,
                     (float2*)a.hb);
  const int64_t nl = cached_launches(a, items, chunk);
  for (int64_t l = 0; l < nl; ++l) {
    a.item0 = items * l / nl;
    const int64_t q = items * (l + 1) / nl - a.item0;
    e = p.dtype == CDD_CI8 ? run_passes<LGN, CDD_CI8, false, GR>(a, q, st)
                           : run_passes<LGN, CDD_CF32, false, GR>(a, q, st);
    if (e) return e;
  }
  return a.fuse ? 0 : launch_integrate(pbuf, P, p.nsamp, p.t_int, p.n_int, p.nchan, st);
}

// exp(+i pi c / L), c < L: the post-twiddle of the packed real inverse.
template <int LG>
static std::vector<float2> make_gsb_pre() {
  const int L = 1 << LG;
  std::vector<float2> t(L);
  for (int c = 0; c < L; ++c) {
    const double ang = M_PI * (double)c / (double)L;
    t[c] = make_float2((float)std::cos(ang), (float)std::sin(ang));
  }
  return t;
}

bool gsb_supported(int nchan) { return nchan >= 128 && nchan <= 2048 && (nchan & (nchan - 1)) == 0; }

template <int LG>
static int launch_gsb_t(const void* spec, int64_t nspec, float* series, void* stream) {
  using SC = typename SubSched<(1 << LG)>::type;
  constexpr int G = SC::T >= 256 ? 1 : 256 / SC::T;
  const float2* tw = nullptr;
  const float2* pre = nullptr;
  int e = twiddles_of<SC>(&tw);
  if (!e) e = cached_table((std::string("gsbpre") + std::to_string(LG)).c_str(),
                           &make_gsb_pre<LG>, &pre);
  if (e) return e;
  const int64_t ngroups = (nspec + G - 1) / G;
  if (ngroups < 1) return (int)hipErrorInvalidValue;
  // as many workgroups as are resident at once (each loops over groups of
  // records): 0.0265 -> 0.0217 ms for the 16,384 records of 512 bins of the
  // 16 MHz full-band workload, against one workgroup per group
  int dev = 0, ncu = 0, per_cu = 0;
  hipError_t he = hipGetDevice(&dev);
  if (he == hipSuccess) he = hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, dev);
  if (he == hipSuccess)
    he = hipOccupancyMaxActiveBlocksPerMultiprocessor(
        &per_cu, reinterpret_cast<const void*>(&gsb_inverse_kernel<SC, G>), SC::T * G, 0);
  if (he != hipSuccess) return (int)he;
  const int64_t nb =
      std::min<int64_t>(ngroups, (int64_t)std::max(ncu, 1) * std::max(per_cu, 1));
  hipLaunchKernelGGL((gsb_inverse_kernel<SC, G>), dim3((unsigned)nb), dim3(SC::T * G), 0,
                     (hipStream_t)stream, (const uint32_t*)spec, (float2*)series, pre, tw, nspec);
  return (int)hipGetLastError();
}

int launch_gsb_inverse(const void* spec, int64_t nspec, int32_t nchan, float* series,
                       void* stream) {
  switch (nchan) {
    case 128: return launch_gsb_t<7>(spec, nspec, series, stream);
    case 256: return launch_gsb_t<8>(spec, nspec, series, stream);
    case 512: return launch_gsb_t<9>(spec, nspec, series, stream);
    case 1024: return launch_gsb_t<10>(spec, nspec, series, stream);
    case 2048: return launch_gsb_t<11>(spec, nspec, series, stream);
  }
  return (int)hipErrorInvalidValue;
}

int64_t fullband_chunk_blocks(const FullbandPlan& f) {
  const int64_t per = std::max<int64_t>(1, kChunkBytes / ((int64_t)(f.N / 2) * 8));
  return std::min(f.nblocks, per);
}

// The row pass forms the chirp itself for records of up to this many blocks:
// a table costs its writing once and its reading in every block (8 bytes per
// bin each, beyond the caches for the long transforms), the FP64 phase about
// 145 clocks per wave of bins, which a pass bound by HBM mostly hides.  At 2^27
// real points, two blocks: table 255 us and row passes of 319 us each.
constexpr int64_t kFlyBlocks = 4;

// gain_of the inverse transform of the records (half a transform pair).
static double gsb_gain(int nchan) {
  switch (nchan) {
    case 128: return 0.5 * gain_of<SubSched<128>::type>();
    case 256: return 0.5 * gain_of<SubSched<256>::type>();
    case 512: return 0.5 * gain_of<SubSched<512>::type>();
    case 1024: return 0.5 * gain_of<SubSched<1024>::type>();
    default: return 0.5 * gain_of<SubSched<2048>::type>();
  }
}

template <int LGN>
static int launch_fullband_t(const FullbandPlan& f, const float* series, float2* S, float* pbuf,
                             float2* hb, float* I, float* vout, void* stream) {
  using SP = Split<LGN>;
  using SR = typename SP::SR;
  constexpr int GR = rows_per_group(SR::T);
  LargeArgs a{};
  int e = set_split<LGN>(a);
  if (e) return e;
  // (half of each mirror pair's power takes two more hardware rotations)
  a.gain = (float)(a.gain + gsb_gain(f.nchan) - kHwRotationGain);
  a.x = series;
  a.S = S;
  a.p = pbuf;
  a.vout = (float2*)vout;
  a.nsamp = f.nsamp / 2;
  a.nblocks = f.nblocks;
  a.nchan = 1;
  a.M = f.M / 2;
  a.nfront = f.nfront / 2;
  a.phase_mode = CDD_PHASE_FP64_REDUCED;
  a.taper = f.taper;
  a.exact_div = 1;
  a.f_lo = f.f_lo;
  a.df = f.bw;
  a.dconst = f.dconst;
  a.dm = f.dm;
  a.P = I;
  a.t_int = f.t_int;
  a.n_int = f.n_int / 2;  // pairs of real samples
  a.fuse = SP::GC % (f.n_int / 2) == 0 ? 1 : 0;
  hipStream_t st = (hipStream_t)stream;
  constexpr int64_t NP = (int64_t)1 << LGN;
  const double dfn = f.bw / (double)NP;
  a.qb = f.dconst * f.dm * dfn * dfn / (f.f_lo * f.f_lo * f.f_lo);
  a.qbeta = dfn / f.f_lo;
  a.hb = f.nblocks <= kFlyBlocks ? nullptr : hb;
  if (a.hb) {
    constexpr int IT = LGN >= 22 ? 4 : 1;
    hipLaunchKernelGGL(band_chirp_table_kernel<IT>, dim3((unsigned)((NP / 2 + 256 * IT - 1) / (256 * IT))),
                       dim3(256), 0, st, a, hb);
  }
  const int64_t nl = cached_launches(a, f.nblocks, fullband_chunk_blocks(f));
  for (int64_t l = 0; l < nl; ++l) {
    a.item0 = f.nblocks * l / nl;
    const int64_t q = f.nblocks * (l + 1) / nl - a.item0;
    if ((e = run_passes<LGN, CDD_CF32, true, GR>(a, q, st))) return e;
  }
  return a.fuse ? 0 : launch_integrate(pbuf, I, f.nsamp / 2, f.t_int, f.n_int / 2, 1, st);
}

int launch_fullband(const FullbandPlan& f, const float* series, void* Sv, float* pbuf,
                    void* Hv, float* I, float* vout, void* stream) {
  float2* S = (float2*)Sv;
  float2* H = (float2*)Hv;
  switch (f.N) {
    case 1 << 16: return launch_fullband_t<15>(f, series, S, pbuf, H, I, vout, stream);
    case 1 << 17: return launch_fullband_t<16>(f, series, S, pbuf, H, I, vout, stream);
    case 1 << 18: return launch_fullband_t<17>(f, series, S, pbuf, H, I, vout, stream);
    case 1 << 19: return launch_fullband_t<18>(f, series, S, pbuf, H, I, vout, stream);
    case 1 << 20: return launch_fullband_t<19>(f, series, S, pbuf, H, I, vout, stream);
    case 1 << 21: return launch_fullband_t<20>(f, series, S, pbuf, H, I, vout, stream);
    case 1 << 22: return launch_fullband_t<21>(f, series, S, pbuf, H, I, vout, stream);
    case 1 << 23: return launch_fullband_t<22>(f, series, S, pbuf, H, I, vout, stream);
    case 1 << 24: return launch_fullband_t<23>(f, series, S, pbuf, H, I, vout, stream);
    case 1 << 25: return launch_fullband_t<24>(f, series, S, pbuf, H, I, vout, stream);
    case 1 << 26: return launch_fullband_t<25>(f, series, S, pbuf, H, I, vout, stream);
    case 1 << 27: return launch_fullband_t<26>(f, series, S, pbuf, H, I, vout, stream);
  }
  return (int)hipErrorInvalidValue;
}

int exact_division_needed(const BeamPlan& p, double dm_abs_max);

int launch_large(const BeamPlan& p, const void* xt, double dm, void* Sv, float* pbuf, float* P,
                 void* vout, void* stream, int32_t* cov_fill, int64_t cov_n) {
  float2* S = (float2*)Sv;
  const int ex = exact_division_needed(p, std::fabs(dm));
  switch (p.N) {
    case 1 << 15: return launch_large_t<15>(p, xt, dm, S, pbuf, P, vout, ex, cov_fill, cov_n, stream);
    case 1 << 16: return launch_large_t<16>(p, xt, dm, S, pbuf, P, vout, ex, cov_fill, cov_n, stream);
    case 1 << 17: return launch_large_t<17>(p, xt, dm, S, pbuf, P, vout, ex, cov_fill, cov_n, stream);
    case 1 << 18: return launch_large_t<18>(p, xt, dm, S, pbuf, P, vout, ex, cov_fill, cov_n, stream);
    case 1 << 19: return launch_large_t<19>(p, xt, dm, S, pbuf, P, vout, ex, cov_fill, cov_n, stream);
    case 1 << 20: return launch_large_t<20>(p, xt, dm, S, pbuf, P, vout, ex, cov_fill, cov_n, stream);
    case 1 << 21: return launch_large_t<21>(p, xt, dm, S, pbuf, P, vout, ex, cov_fill, cov_n, stream);
    case 1 << 22: return launch_large_t<22>(p, xt, dm, S, pbuf, P, vout, ex, cov_fill, cov_n, stream);
    case 1 << 23: return launch_large_t<23>(p, xt, dm, S, pbuf, P, vout, ex, cov_fill, cov_n, stream);
    case 1 << 24: return launch_large_t<24>(p, xt, dm, S, pbuf, P, vout, ex, cov_fill, cov_n, stream);
    case 1 << 25: return launch_large_t<25>(p, xt, dm, S, pbuf, P, vout, ex, cov_fill, cov_n, stream);
    case 1 << 26: return launch_large_t<26>(p, xt, dm, S, pbuf, P, vout, ex, cov_fill, cov_n, stream);
  }
  return (int)hipErrorInvalidValue;
}

}  // namespace cdd
