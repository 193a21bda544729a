// Layout change, channel delays and the delay-aligned channel sum.
#include <hip/hip_runtime.h>

#include <cmath>
#include <type_traits>

#include "cdd_fft.h"
#include "cdd_internal.h"
#include "cdd_rules.h"

namespace cdd {

// Delay of channel c at one DM in integrated samples (the expression of
// delays_kernel below and of the host planner, in the same order, without
// fused multiply-adds, so all three round to the same integers).
__device__ __forceinline__ int32_t channel_delay(int c, double dm, int32_t nchan, double f_centre,
                                                 double bw, double df, double dconst,
                                                 int32_t n_int) {
#pragma clang fp contract(off)
  const double fc = (f_centre - bw / 2.0) + ((double)c + 0.5) * df;
  const int cref = dm >= 0 ? nchan - 1 : 0;
  const double fref = (f_centre - bw / 2.0) + ((double)cref + 0.5) * df;
  const double x = dconst * dm * (1.0 / (fc * fc) - 1.0 / (fref * fref)) * df / (double)n_int;
  return (int32_t)floor(x + 0.5);
}

// One DM's channel delays, computed by one workgroup of the layout change.
struct DelayArgs {
  int32_t* d;  // null: none
  double dm, f_centre, bw, df, dconst;
  int32_t nchan, n_int;
};

static DelayArgs delay_args(const BeamPlan& p, double dm, int32_t* delays) {
  DelayArgs dl{};
  if (delays) {
    dl.d = delays;
    dl.dm = dm;
    dl.f_centre = p.f_centre;
    dl.bw = p.bw;
    dl.df = p.df;
    dl.dconst = p.dconst;
    dl.nchan = p.nchan;
    dl.n_int = p.n_int;
  }
  return dl;
}

// ---------------------------------------------------------------------------
// Time-major [nsamp][nchan] -> channel-major [nchan][nsamp].
// int8 pairs (2 bytes per complex sample): 64 samples x 128 channels per
// workgroup through LDS; each lane moves 8 bytes (4 complex samples) on both
// the load (along channels) and the store (along time) side.
// ---------------------------------------------------------------------------
// With ct.H set, workgroup w < ct.nwg also writes table workgroup w's share
// of the one-DM chirp table once its tile stores are issued: the table's
// FP64 arithmetic runs while the memory-bound layout change's traffic is in
// flight, instead of in a kernel of its own beside it.  With dl.d set, the
// last workgroup also writes the channel delays.
__device__ __forceinline__ void table_and_delays(const ChirpTableArgs& ct, const DelayArgs& dl,
                                                 int l) {
  if (ct.H != nullptr && blockIdx.x < ct.nwg) chirp_table_part(ct, blockIdx.x, l);
  if (dl.d != nullptr && blockIdx.x == gridDim.x - 1)
    for (int c = l; c < dl.nchan; c += 256)
      dl.d[c] = channel_delay(c, dl.dm, dl.nchan, dl.f_centre, dl.bw, dl.df, dl.dconst, dl.n_int);
}

__global__ __launch_bounds__(256) void transpose_i8_kernel(const unsigned short* __restrict__ in,
                                                           unsigned short* __restrict__ out,
                                                           int64_t nsamp, int32_t nchan,
                                                           int32_t tiles_c, int32_t in_aligned,
                                                           int64_t ostr, const ChirpTableArgs ct,
                                                           const DelayArgs dl) {
  __shared__ unsigned short tile[64][128 + 4];
  const int64_t bid = blockIdx.x;
  const int c0 = (int)(bid % tiles_c) * 128;
  const int64_t t0 = (bid / tiles_c) * 64;
  const int l = threadIdx.x;
  const bool full =
      in_aligned && (c0 + 128 <= nchan) && (t0 + 64 <= nsamp) && (nchan % 4 == 0);
  // load: 32 lanes per row, 4 channels each; 8 rows per pass of 256 lanes
  {
    const int cl = (l & 31) * 4, rl = l >> 5;
#pragma unroll
    for (int i = 0; i < 64; i += 8) {
      const int r = rl + i;
      const int64_t ts = t0 + r;
      if (full) {
        const uint2 w = *(const uint2*)(in + ts * nchan + c0 + cl);
        tile[r][cl + 0] = (unsigned short)(w.x & 0xffff);
        tile[r][cl + 1] = (unsigned short)(w.x >> 16);
        tile[r][cl + 2] = (unsigned short)(w.y & 0xffff);
        tile[r][cl + 3] = (unsigned short)(w.y >> 16);
      } else {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int cs = c0 + cl + q;
          tile[r][cl + q] = (ts < nsamp && cs < nchan) ? in[ts * nchan + cs] : (unsigned short)0;
        }
      }
    }
  }
  __syncthreads();
  // store: 16 lanes per channel row, 4 samples each; 16 channels per pass
  {
    const int tl = (l & 15) * 4, cr = l >> 4;
#pragma unroll
    for (int i = 0; i < 128; i += 16) {
      const int c = cr + i;
      const int cs = c0 + c;
      if (cs >= nchan) continue;
      const int64_t ts = t0 + tl;
      if (full || ts + 4 <= nsamp) {
        if ((nsamp & 3) == 0 || full) {
          uint2 w;
          w.x = (unsigned)tile[tl + 0][c] | ((unsigned)tile[tl + 1][c] << 16);
          w.y = (unsigned)tile[tl + 2][c] | ((unsigned)tile[tl + 3][c] << 16);
          if (((int64_t)cs * ostr + ts) % 4 == 0) {
            *(uint2*)(out + (int64_t)cs * ostr + ts) = w;
            continue;
          }
        }
      }
#pragma unroll
      for (int q = 0; q < 4; ++q)
        if (ts + q < nsamp) out[(int64_t)cs * ostr + ts + q] = tile[tl + q][c];
    }
  }
  table_and_delays(ct, dl, l);
}

// Float pairs: tiles of kTileT samples by 64 channels, bound by memory.  101
// channels of 40,001 samples (65 MB moved): 18.2 us with 64-sample tiles (33 KB
// of LDS, four workgroups per CU), 14.6 us with 32, which keep twice as many
// workgroups in different phases.  The chirp table and the delays ride along as
// above: with them in kernels of their own a pass over that record took 61 us,
// now 41.
constexpr int kTileT = 32;
__global__ __launch_bounds__(256) void transpose_c8_kernel(const float2* __restrict__ in,
                                                           float2* __restrict__ out,
                                                           int64_t nsamp, int32_t nchan,
                                                           int32_t tiles_c, int64_t ostr,
                                                           const ChirpTableArgs ct,
                                                           const DelayArgs dl) {
  __shared__ float2 tile[kTileT][65];
  const int64_t bid = blockIdx.x;
  const int c0 = (int)(bid % tiles_c) * 64;
  const int64_t t0 = (bid / tiles_c) * kTileT;
  {
    const int tx = threadIdx.x & 63, ty = threadIdx.x >> 6;
    const int cs = c0 + tx;
#pragma unroll
    for (int i = 0; i < kTileT; i += 4) {
      const int64_t ts = t0 + ty + i;
      if (ts < nsamp && cs < nchan) tile[ty + i][tx] = in[ts * nchan + cs];
    }
  }
  __syncthreads();
  {
    const int tx = threadIdx.x % kTileT, ty = threadIdx.x / kTileT;
    const int64_t ts = t0 + tx;
#pragma unroll
    for (int i = 0; i < 64; i += 256 / kTileT) {
      const int cs = c0 + ty + i;
      if (cs < nchan && ts < nsamp) out[(int64_t)cs * ostr + ts] = tile[tx][ty + i];
    }
  }
  table_and_delays(ct, dl, threadIdx.x);
}

// Tiles of the layout change.
static int64_t transpose_tiles(int32_t dtype, int64_t nsamp, int32_t nchan, int64_t* tiles_c) {
  const int tc = dtype == CDD_CI8 ? 128 : 64, tt = dtype == CDD_CI8 ? 64 : kTileT;
  *tiles_c = (nchan + tc - 1) / tc;
  return *tiles_c * ((nsamp + tt - 1) / tt);
}

static int launch_tiles(const void* in, void* out, int32_t dtype, int64_t nsamp, int32_t nchan,
                        int64_t out_stride, const ChirpTableArgs& ct, const DelayArgs& dl,
                        hipStream_t st) {
  int64_t tiles_c = 0;
  const int64_t n = transpose_tiles(dtype, nsamp, nchan, &tiles_c);
  if (n <= 0 || n > 0x7fffffffLL) return (int)hipErrorInvalidValue;
  if (dtype == CDD_CI8)
    hipLaunchKernelGGL(transpose_i8_kernel, dim3((unsigned)n), dim3(256), 0, st,
                       (const unsigned short*)in, (unsigned short*)out, nsamp, nchan,
                       (int32_t)tiles_c, (int32_t)(((uintptr_t)in & 7u) == 0), out_stride, ct, dl);
  else
    hipLaunchKernelGGL(transpose_c8_kernel, dim3((unsigned)n), dim3(256), 0, st,
                       (const float2*)in, (float2*)out, nsamp, nchan, (int32_t)tiles_c,
                       out_stride, ct, dl);
  return (int)hipGetLastError();
}

int launch_transpose(const void* in, void* out, int32_t dtype, int64_t nsamp, int32_t nchan,
                     int64_t out_stride, void* stream) {
  return launch_tiles(in, out, dtype, nsamp, nchan, out_stride, ChirpTableArgs{}, DelayArgs{},
                      (hipStream_t)stream);
}

bool transpose_chirp_fits(const BeamPlan& p) {
  if (p.nchan < 2 || !block_supported(p.N)) return false;
  int64_t tiles_c = 0;
  // at least one channel's table per workgroup at kpt = N/256
  return (int64_t)p.nchan <= transpose_tiles(p.dtype, p.nsamp, p.nchan, &tiles_c);
}

int launch_transpose_chirp(const BeamPlan& p, const void* in, void* out, double dm, void* H,
                           void* stream, int32_t* delays, int variant) {
  if (!transpose_chirp_fits(p) || H == nullptr) return (int)hipErrorInvalidValue;
  int64_t tiles_c = 0;
  const int64_t n = transpose_tiles(p.dtype, p.nsamp, p.nchan, &tiles_c);
  // the fewest table entries per thread that the layout change's workgroups cover
  int kpt = 1;
  while ((int64_t)p.nchan * (p.N / (256 * kpt)) > n && 256 * kpt * 2 <= p.N) kpt *= 2;
  return launch_tiles(in, out, p.dtype, p.nsamp, p.nchan, xt_stride(p),
                      chirp_table_args(p, dm, H, kpt, variant), delay_args(p, dm, delays),
                      (hipStream_t)stream);
}

// ---------------------------------------------------------------------------
// Channel delays in FP64 (Sec. 1.2; the linear term of Eq. 2): the same
// operations, in the same order and without fused multiply-adds, as the
// host planner, so both round to the same integers.
// ---------------------------------------------------------------------------
#pragma clang fp contract(off)
__global__ __launch_bounds__(256) void delays_kernel(int32_t* __restrict__ d, DmTile dms,
                                                     int32_t nchan, double f_centre, double bw,
                                                     double df, double dconst, int32_t n_int) {
  const int c = blockIdx.x * 256 + threadIdx.x;
  const int i = blockIdx.y;
  if (c >= nchan || i >= dms.ndm) return;
  d[(int64_t)i * nchan + c] =
      channel_delay(c, dms.dm[i], nchan, f_centre, bw, df, dconst, n_int);
}
#pragma clang fp contract(on)

int launch_delays(const BeamPlan& p, const DmTile& dms, int32_t* d, void* stream) {
  dim3 grid((unsigned)((p.nchan + 255) / 256), (unsigned)dms.ndm);
  hipLaunchKernelGGL(delays_kernel, grid, dim3(256), 0, (hipStream_t)stream, d, dms, p.nchan,
                     p.f_centre, p.bw, p.df, p.dconst, p.n_int);
  return (int)hipGetLastError();
}

// v[i] = x for i < n (four per thread).
__global__ __launch_bounds__(256) void fill_i32_kernel(int32_t* __restrict__ v, int64_t n,
                                                       int32_t x) {
  const int64_t i = ((int64_t)blockIdx.x * 256 + threadIdx.x) * 4;
#pragma unroll
  for (int j = 0; j < 4; ++j)
    if (i + j < n) v[i + j] = x;
}

int launch_fill_i32(int32_t* v, int64_t n, int32_t x, void* stream) {
  if (n <= 0) return 0;
  const int64_t nb = (n + 1023) / 1024;
  if (nb > 0x7fffffffLL) return (int)hipErrorInvalidValue;
  hipLaunchKernelGGL(fill_i32_kernel, dim3((unsigned)nb), dim3(256), 0, (hipStream_t)stream, v,
                     n, x);
  return (int)hipGetLastError();
}

// ---------------------------------------------------------------------------
// Detection and integration without the coherent step (incoherent
// dedispersion): P[c][u] = sum over r < n_int of |x_c[u n_int + r]|^2, in
// order; consecutive threads take consecutive u of one channel.
// ---------------------------------------------------------------------------
template <int DT>
__global__ __launch_bounds__(256) void detect_kernel(const void* __restrict__ xt,
                                                     float* __restrict__ P, int64_t xstride,
                                                     int64_t t_int, int32_t n_int) {
  const int64_t u = (int64_t)blockIdx.x * 256 + threadIdx.x;
  const int c = blockIdx.y;
  if (u >= t_int) return;
  float s = 0.f;
  const int64_t base = (int64_t)c * xstride + u * n_int;
  for (int r = 0; r < n_int; ++r) {
    float re, im;
    if constexpr (DT == CDD_CI8) {
      const unsigned short w = ((const unsigned short*)xt)[base + r];
      re = (float)(signed char)(w & 0xff);
      im = (float)(signed char)(w >> 8);
    } else {
      const float2 z = ((const float2*)xt)[base + r];
      re = z.x;
      im = z.y;
    }
    s += re * re + im * im;
  }
  P[(int64_t)c * t_int + u] = s;
}

int launch_detect(const BeamPlan& p, const void* xt, float* P, void* stream) {
  const int64_t nb = (p.t_int + 255) / 256;
  if (nb <= 0) return 0;
  if (nb > 0x7fffffffLL || p.nchan > 65535) return (int)hipErrorInvalidValue;
  dim3 grid((unsigned)nb, (unsigned)p.nchan);
  if (p.dtype == CDD_CI8)
    hipLaunchKernelGGL(detect_kernel<CDD_CI8>, grid, dim3(256), 0, (hipStream_t)stream, xt, P,
                       xt_stride(p), p.t_int, p.n_int);
  else
    hipLaunchKernelGGL(detect_kernel<CDD_CF32>, grid, dim3(256), 0, (hipStream_t)stream, xt, P,
                       xt_stride(p), p.t_int, p.n_int);
  return (int)hipGetLastError();
}

// The same straight from the time-major record, without a channel-major copy:
// a workgroup takes 32 outputs of a run of CH = 32 CPT (or 64) channels, each
// lane the n_int samples of CPT adjacent channels, and turns the sums through
// LDS so that both sides are whole runs (CH samples in, 32 floats out).  It is
// bound by HBM: the record is read once and P written once, where the copy
// read and wrote the record again (512 channels x 250,000 int8 samples, n_int
// 4: 92 + 118 us for copy and detection, 76 us here).  NI: n_int at compile
// time (0: any).  The last workgroup also writes the channel delays.  Where the
// copy and detect_kernel are taken instead: detect_from_record.
template <int DT, int CPT, int NI>
__global__ __launch_bounds__(256) void detect_tiled_kernel(const void* __restrict__ in,
                                                           float* __restrict__ P, int32_t nchan,
                                                           int32_t tiles_c, int64_t t_int,
                                                           int32_t n_int_, const DelayArgs dl) {
  constexpr int LC = CPT == 1 ? 64 : 32;   // lanes along channels
  constexpr int CH = LC * CPT;             // channels per workgroup
  constexpr int UP = 256 / LC, U = 32;     // outputs per step and per workgroup
  __shared__ float tile[U][CH + 1];
  const int n_int = NI ? NI : n_int_;
  const int c0 = (int)(blockIdx.x % tiles_c) * CH;
  const int64_t u0 = (int64_t)(blockIdx.x / tiles_c) * U;
  const int cl = ((int)threadIdx.x % LC) * CPT, ul = threadIdx.x / LC;
  const bool in_c = c0 + cl < nchan;  // (CPT divides nchan)
#pragma unroll
  for (int i = 0; i < U / UP; ++i) {
    const int64_t u = u0 + ul + i * UP;
    float acc[CPT];
#pragma unroll
    for (int q = 0; q < CPT; ++q) acc[q] = 0.f;
    if (in_c && u < t_int) {
      const int64_t at = u * n_int * nchan + c0 + cl;
      auto add = [&](int r) {
        if constexpr (DT == CDD_CF32) {
          const float2 z = ((const float2*)in)[at + (int64_t)r * nchan];
          acc[0] += z.x * z.x + z.y * z.y;
        } else {
          unsigned w[(CPT + 1) / 2];
          if constexpr (CPT == 4) {
            const uint2 x = *(const uint2*)((const unsigned short*)in + at + (int64_t)r * nchan);
            w[0] = x.x;
            w[1] = x.y;
          } else {
            w[0] = ((const unsigned short*)in)[at + (int64_t)r * nchan];
          }
#pragma unroll
          for (int q = 0; q < CPT; ++q) {
            const unsigned h = w[q / 2] >> (16 * (q & 1));
            const float re = (float)(signed char)(h & 0xff);
            const float im = (float)(signed char)((h >> 8) & 0xff);
            acc[q] += re * re + im * im;
          }
        }
      };
      if constexpr (NI > 0) {
#pragma unroll
        for (int r = 0; r < NI; ++r) add(r);
      } else {
#pragma unroll 4
        for (int r = 0; r < n_int; ++r) add(r);
      }
    }
#pragma unroll
    for (int q = 0; q < CPT; ++q) tile[ul + i * UP][cl + q] = acc[q];
  }
  __syncthreads();
  // 32 lanes per channel row
  const int us = threadIdx.x & 31;
  for (int c = threadIdx.x >> 5; c < CH && c0 + c < nchan; c += 8)
    if (u0 + us < t_int) P[(int64_t)(c0 + c) * t_int + u0 + us] = tile[us][c];
  if (dl.d != nullptr && blockIdx.x == gridDim.x - 1)
    for (int c = threadIdx.x; c < dl.nchan; c += 256)
      dl.d[c] = channel_delay(c, dl.dm, dl.nchan, dl.f_centre, dl.bw, dl.df, dl.dconst, dl.n_int);
}

bool detect_tiled_fits(const BeamPlan& p) {
  if (!detect_from_record(p.dtype == CDD_CF32, p.nchan, p.nsamp, p.n_int)) return false;
  return ((int64_t)(p.nchan + 63) / 64) * ((p.t_int + 31) / 32) <= 0x7fffffffLL;
}

template <int DT, int CPT>
static void detect_tiled_launch(const BeamPlan& p, const void* in, float* P, const DelayArgs& dl,
                                hipStream_t st) {
  constexpr int CH = CPT == 1 ? 64 : 32 * CPT;
  const int32_t tc = (p.nchan + CH - 1) / CH;
  const dim3 grid((unsigned)(tc * ((p.t_int + 31) / 32))), block(256);
  auto go = [&](auto NI) {
    hipLaunchKernelGGL((detect_tiled_kernel<DT, CPT, decltype(NI)::value>), grid, block, 0, st,
                       in, P, p.nchan, tc, p.t_int, p.n_int, dl);
  };
  switch (p.n_int) {
    case 1: return go(std::integral_constant<int, 1>{});
    case 2: return go(std::integral_constant<int, 2>{});
    case 4: return go(std::integral_constant<int, 4>{});
    case 8: return go(std::integral_constant<int, 8>{});
    default: return go(std::integral_constant<int, 0>{});
  }
}

int launch_detect_tiled(const BeamPlan& p, const void* in, float* P, double dm, int32_t* delays,
                        void* stream) {
  if (!detect_tiled_fits(p)) return (int)hipErrorInvalidValue;
  const DelayArgs dl = delay_args(p, dm, delays);
  hipStream_t st = (hipStream_t)stream;
  if (p.dtype == CDD_CF32)
    detect_tiled_launch<CDD_CF32, 1>(p, in, P, dl, st);
  else if (p.nchan % 4 == 0 && ((uintptr_t)in & 7u) == 0)
    detect_tiled_launch<CDD_CI8, 4>(p, in, P, dl, st);  // rows of whole 8-byte words
  else
    detect_tiled_launch<CDD_CI8, 1>(p, in, P, dl, st);
  return (int)hipGetLastError();
}

// ---------------------------------------------------------------------------
// Folding at a known period: L threads per phase bin b.  Sample u lies in
// period floor(u/period + phase0) and in bin floor(frac(...) * nbins) of it
// (FP64, contraction off, clamped to nbins - 1).  Thread l of a bin takes the
// periods k = l, l + L, ...: it visits the samples around
// [(k + b/nbins - phase0) period, (k + (b+1)/nbins - phase0) period) and adds
// those of that period and bin in FP64; the L sums are added pairwise (a fixed
// order) and rounded to FP32 once.  With one thread per bin the periods were a
// serial chain of dependent FP64 divisions and loads (62,500 samples into 256
// bins: 78 us; 15,625: 25 us).  Where one thread has a bin to itself it goes on
// from the samples already visited, so that the margins of neighbouring periods
// are not visited twice, and any period of the sample's bin counts (1,000,000
// samples into 8193 bins at 1.5 samples a period: 241 ms, 500 with the margins).
// ---------------------------------------------------------------------------
#pragma clang fp contract(off)
template <int L>
__global__ __launch_bounds__(256) void fold_kernel(const float* __restrict__ I, int64_t t_int,
                                                   double period, double phase0, int32_t nbins,
                                                   float* __restrict__ prof,
                                                   int32_t* __restrict__ cnt) {
  __shared__ double ss[256];
  __shared__ int32_t sn[256];
  const int t = threadIdx.x, l = t % L;
  const int64_t b = (int64_t)blockIdx.x * (256 / L) + t / L;
  double s = 0.0;
  int32_t n = 0;
  if (b < nbins) {
    const int64_t k0 = (int64_t)floor(phase0) - 1;
    const int64_t k1 = (int64_t)floor((double)(t_int - 1) / period + phase0) + 1;
    int64_t next = 0;  // (L == 1) samples below have been visited
    for (int64_t k = k0 + l; k <= k1; k += L) {
      const double lo = ((double)k + (double)b / nbins - phase0) * period;
      const double hi = ((double)k + (double)(b + 1) / nbins - phase0) * period;
      int64_t u0 = (int64_t)floor(lo) - 2, u1 = (int64_t)ceil(hi) + 2;
      if (u0 < next) u0 = next;
      if (u1 > t_int) u1 = t_int;
      for (int64_t u = u0; u < u1; ++u) {
        const double x = (double)u / period + phase0;
        const double fl = floor(x);
        const int q = (int)floor((x - fl) * (double)nbins);
        if ((L == 1 || (int64_t)fl == k) && (q < nbins ? q : nbins - 1) == b) {
          s += (double)I[u];
          ++n;
        }
      }
      if (L == 1 && u1 > next) next = u1;
    }
  }
  if constexpr (L > 1) {
    ss[t] = s;
    sn[t] = n;
    __syncthreads();
#pragma unroll
    for (int d = L / 2; d > 0; d /= 2) {
      if (l < d) {
        s += ss[t + d];
        n += sn[t + d];
        ss[t] = s;
        sn[t] = n;
      }
      __syncthreads();
    }
  }
  if (l == 0 && b < nbins) {
    prof[b] = (float)s;
    if (cnt) cnt[b] = n;
  }
}
#pragma clang fp contract(on)

template <int L>
static int fold_launch(const float* I, int64_t t_int, double period, double phase0, int32_t nbins,
                       float* profile, int32_t* counts, hipStream_t st) {
  const int64_t nb = ((int64_t)nbins * L + 255) / 256;
  if (nb <= 0 || nb > 0x7fffffffLL) return (int)hipErrorInvalidValue;
  hipLaunchKernelGGL((fold_kernel<L>), dim3((unsigned)nb), dim3(256), 0, st, I, t_int, period,
                     phase0, nbins, profile, counts);
  return (int)hipGetLastError();
}

int launch_fold(const float* I, int64_t t_int, double period, double phase0, int32_t nbins,
                float* profile, int32_t* counts, void* stream) {
  hipStream_t st = (hipStream_t)stream;
  switch (fold_threads(t_int, period, nbins)) {
    case 256: return fold_launch<256>(I, t_int, period, phase0, nbins, profile, counts, st);
    case 64: return fold_launch<64>(I, t_int, period, phase0, nbins, profile, counts, st);
    default: return fold_launch<1>(I, t_int, period, phase0, nbins, profile, counts, st);
  }
}

// ---------------------------------------------------------------------------
// I[u] = sum over channels c with u + d_c < T_int of P_c[u + d_c], cov[u] =
// number of terms.  A workgroup covers 64 consecutive u; its G waves each sum
// a contiguous channel range in ascending order, and the G partial sums are
// added in ascending wave order -- a fixed order, no atomics, so results do
// not depend on scheduling.  grid.y = DM trial.
// Each channel row is read through a buffer resource whose range ends at
// src_lim: a term past the end is pointed at src_lim itself and reads as zero
// (adding +0 leaves the sum unchanged), so the loads carry no branch; eight
// channels' loads are issued before they are added.  Rows of 2^29 floats or
// more take the checked loop.
// ---------------------------------------------------------------------------
template <int G, bool BUF>
__global__ __launch_bounds__(64 * G) void dsum_kernel(const float* __restrict__ P,
                                                      const int32_t* __restrict__ d,
                                                      float* __restrict__ I,
                                                      int32_t* __restrict__ cov, int32_t nchan,
                                                      int64_t p_stride, int64_t p_dm_stride,
                                                      int64_t src_lim, int64_t u_begin,
                                                      int64_t u_count, int64_t out_stride) {
  __shared__ float ps[G][64];
  __shared__ int32_t pn[G][64];
  const int i = blockIdx.y;
  const int lane = threadIdx.x & 63;
  const int g = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);  // wave index (uniform)
  const int64_t uo = (int64_t)blockIdx.x * 64 + lane;
  const int64_t u = u_begin + uo;
  const float* Pi = P + (int64_t)i * p_dm_stride;
  const int32_t* di = d + (int64_t)i * nchan;
  const int per = (nchan + G - 1) / G;
  const int c_lo = g * per, c_hi = min(nchan, c_lo + per);
  float acc = 0.f;
  int32_t n = 0;
  if constexpr (BUF) {
    // lanes past u_count read offset 0 (in range or zero) and are not stored
    const bool live = uo < u_count;
    const int ub = live ? (int)u : 0;
    const int lim = (int)src_lim;
    int c = c_lo;
    for (; c + 8 <= c_hi; c += 8) {
      float x[8];
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
            (void*)(Pi + (int64_t)(c + j) * p_stride), (short)0, lim * 4, 0x00020000);
        const int64_t src = (int64_t)ub + di[c + j];
        const bool in = src < lim;
        x[j] = __builtin_bit_cast(
            float, __builtin_amdgcn_raw_buffer_load_b32(rs, (in ? (int)src : lim) * 4, 0, 0));
        n += in;
      }
#pragma unroll
      for (int j = 0; j < 8; ++j) acc += x[j];
    }
    for (; c < c_hi; ++c) {
      const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
          (void*)(Pi + (int64_t)c * p_stride), (short)0, lim * 4, 0x00020000);
      const int64_t src = (int64_t)ub + di[c];
      const bool in = src < lim;
      acc += __builtin_bit_cast(
          float, __builtin_amdgcn_raw_buffer_load_b32(rs, (in ? (int)src : lim) * 4, 0, 0));
      n += in;
    }
  } else {
    if (uo < u_count) {
      for (int c = c_lo; c < c_hi; ++c) {
        const int64_t src = u + di[c];
        if (src < src_lim) {
          acc += Pi[(int64_t)c * p_stride + src];
          ++n;
        }
      }
    }
  }
  ps[g][lane] = acc;
  pn[g][lane] = n;
  __syncthreads();
  if (g == 0 && uo < u_count) {
    float s = ps[0][lane];
    int32_t m = pn[0][lane];
#pragma unroll
    for (int k = 1; k < G; ++k) {
      s += ps[k][lane];
      m += pn[k][lane];
    }
    I[(int64_t)i * out_stride + uo] = s;
    if (cov) cov[(int64_t)i * out_stride + uo] = m;
  }
}

template <int G>
static void dsum_launch(bool buf, dim3 grid, hipStream_t st, const float* P, const int32_t* d,
                        float* I, int32_t* cov, int nchan, int64_t p_stride, int64_t p_dm_stride,
                        int64_t src_lim, int64_t u_begin, int64_t u_count, int64_t out_stride) {
  if (buf)
    hipLaunchKernelGGL((dsum_kernel<G, true>), grid, dim3(64 * G), 0, st, P, d, I, cov, nchan,
                       p_stride, p_dm_stride, src_lim, u_begin, u_count, out_stride);
  else
    hipLaunchKernelGGL((dsum_kernel<G, false>), grid, dim3(64 * G), 0, st, P, d, I, cov, nchan,
                       p_stride, p_dm_stride, src_lim, u_begin, u_count, out_stride);
}

int launch_dsum_range(int nchan, int ndm, const float* P, int64_t p_stride, int64_t p_dm_stride,
                      int64_t src_lim, int64_t u_begin, int64_t u_count, const int32_t* d,
                      float* I, int32_t* cov, int64_t out_stride, void* stream) {
  if (u_count <= 0) return 0;
  const int64_t nb = (u_count + 63) / 64;
  if (nb > 0x7fffffffLL || ndm < 1 || ndm > 65535) return (int)hipErrorInvalidValue;
  dim3 grid((unsigned)nb, (unsigned)ndm);
  hipStream_t st = (hipStream_t)stream;
  // 32-bit byte offsets: row lengths and output positions below 2^29
  const bool buf = src_lim >= 0 && src_lim < (1LL << 29) && u_begin + u_count < (1LL << 29);
  if (nchan >= 256)
    dsum_launch<16>(buf, grid, st, P, d, I, cov, nchan, p_stride, p_dm_stride, src_lim, u_begin,
                    u_count, out_stride);
  else if (nchan >= 64)
    dsum_launch<8>(buf, grid, st, P, d, I, cov, nchan, p_stride, p_dm_stride, src_lim, u_begin,
                   u_count, out_stride);
  else
    dsum_launch<1>(buf, grid, st, P, d, I, cov, nchan, p_stride, p_dm_stride, src_lim, u_begin,
                   u_count, out_stride);
  return (int)hipGetLastError();
}

int launch_dsum(const BeamPlan& p, int ndm, const float* P, const int32_t* d, float* I,
                int32_t* cov, int64_t out_stride, void* stream) {
  return launch_dsum_range(p.nchan, ndm, P, p.t_int, (int64_t)p.nchan * p.t_int, p.t_int, 0,
                           p.t_int, d, I, cov, out_stride, stream);
}

}  // namespace cdd
