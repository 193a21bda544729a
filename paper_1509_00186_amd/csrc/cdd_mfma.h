// The first forward pass of the block kernels on the matrix cores (8-bit records).
//
// A DFT of 16 complex points is a real 32 x 32 matrix F acting on columns of
// 32 values (re, im interleaved), so 32 butterflies are one 32 x 32 x 32
// product: two v_mfma_f32_32x32x16_f16.  8-bit samples are exact in a half; F is
// carried as a pair of halves, Fh + Fl, of kMfScale F.  A pair holds 22 bits, two
// fewer than FP32 for the worst entries (sin(pi/8) would be 2.4e-8 off, 6e-9 as an
// FP32 number); the scale is one at which all eight magnitudes cos(k pi/16) happen
// to lie close to pairs: the largest error is 1.4e-9, every entry at or below that of
// its FP32 number, and none of the parts is a subnormal.  (Three halves without a
// scale: 512 channels 413 -> 428 us.)  The scale is taken out by the chirp, with the
// 1/N of the inverse transform.  The products accumulate in FP32.
//
// The pass takes three vector operations per sample (byte pair to halves) where the
// conversion and the radix-16 butterfly took 14, and the matrix cores, idle
// otherwise, work beside the vector ALU, which bounds these kernels.  The later
// passes stay on the vector ALU: their FP32 values would have to be split into
// two halves, six vector operations and three products for ten operations saved
// (512 channels: 0.62 ms and more for the call, against 0.43).
//
// Lane layout.  Lanes l and l + 32 of a wave share a butterfly column: half
// h = l / 32 holds the points r = 8 a + 4 h + b (a < 2, b < 4) on input (the
// K index of the two products) and, by the order of F's rows, the same set on
// output.  A wave's 64 columns are two tiles of 32, the even and the odd ones,
// so a lane's samples come in neighbouring pairs, two to a 4-byte load.
// Radix 32: X[k], X[k + 16] = E[k] +- O[k] over even and odd inputs, O with
// its own matrix W32^(k (2r + 1)).
#pragma once

#include "cdd_fft.h"

namespace cdd {

typedef _Float16 half2v __attribute__((ext_vector_type(2)));
typedef _Float16 half8v __attribute__((ext_vector_type(8)));
typedef float float16v __attribute__((ext_vector_type(16)));
typedef unsigned int uint4v __attribute__((ext_vector_type(4)));

template <class S>
constexpr bool mf_schedule() {
  // with 16 points a thread the fragments' loads cost what the pass saves
  // (N 2048: 3.00 ms for the four beams against 2.86 without)
  return (S::rad_f(0) == 16 || S::rad_f(0) == 32) && S::E >= 32;
}

// Matrix fragments: operand A of the 32 x 32 x 16 product, lane l holding row
// l % 32 and the eight columns 8 (l / 32) + e.  Row 2m + c is component c of
// output k(m), k(m) = m with its two middle bits exchanged (so that half h
// receives k = 8 a + 4 h + b); column 16 s + 8 h + e is component e % 2 of
// input r = 8 s + 4 h + e / 2.  Kinds: 0 exp(-2 pi i r k/16); 1 (odd inputs of
// radix 32) exp(-2 pi i k (2r + 1)/32).  Fragment order: kind, s, part (largest
// first); 64 lanes of 16 bytes each.
enum { kMfPlain = 0, kMfOdd = 1, kMfKinds = 2 };
constexpr int kMfParts = 2;
constexpr float kMfScale = 4154.09765625f;
inline std::vector<float2> make_mf_table() {
  std::vector<float2> out((size_t)kMfKinds * 2 * kMfParts * 64 * 2);  // 16 bytes per lane
  _Float16* h = (_Float16*)out.data();
  for (int kind = 0; kind < kMfKinds; ++kind)
    for (int s = 0; s < 2; ++s)
      for (int l = 0; l < 64; ++l)
        for (int e = 0; e < 8; ++e) {
          const int row = l & 31, m = row >> 1, c = row & 1;
          const int k = (m & 9) | ((m & 2) << 1) | ((m & 4) >> 1);
          const int r = 8 * s + 4 * (l >> 5) + (e >> 1), ci = e & 1;
          const int num = kind == kMfPlain ? 2 * r * k : k * (2 * r + 1);
          const double ang = -2.0 * M_PI * (double)(num % 32) / 32.0;
          const double re = std::cos(ang), im = std::sin(ang);
          // out_re = re x_re - im x_im, out_im = im x_re + re x_im
          const double v = c == ci ? re : c ? im : -im;
          const double z = std::fabs(v) < 1e-9 ? 0.0 : v;
          double rest = z * (double)kMfScale;
          for (int p = 0; p < kMfParts; ++p) {
            const _Float16 part = (_Float16)rest;
            rest -= (double)part;
            h[(((size_t)(kind * 2 + s) * kMfParts + p) * 64 + l) * 8 + e] = part;
          }
        }
  return out;
}

struct MfMat {
  half8v part[kMfParts][2];
};
__device__ __forceinline__ MfMat mf_matrix(const float2* tab, int kind, int lane) {
  MfMat m;
  const auto p = gptr((const uint4v*)tab);
#pragma unroll
  for (int i = 0; i < kMfParts; ++i)
#pragma unroll
    for (int s = 0; s < 2; ++s)
      m.part[i][s] =
          __builtin_bit_cast(half8v, p[((kind * 2 + s) * kMfParts + i) * 64 + lane]);
  return m;
}

// Element idx of a thread in the first pass (radix R): point thread_r(t) +
// rc_in(idx) of the butterfly in column thread_col(t) + cc(idx), and after the
// butterflies output thread_r_out(t) + rc_out(idx) of the same column.
// Thread and constant parts occupy disjoint bits.
template <class S, int R>
struct MfMap {
  static constexpr int PT = R / 2;  // points per tile and thread
  static __device__ __forceinline__ int thread_col(int t) { return (t & ~63) | ((t & 31) << 1); }
  static __device__ __forceinline__ int thread_r_in(int t) {
    return ((t >> 5) & 1) * (R == 32 ? 8 : 4);
  }
  static __device__ __forceinline__ int thread_r_out(int t) { return ((t >> 5) & 1) * 4; }
  static constexpr int cc(int idx) {
    return ((idx / PT) & 1) + S::T * ((idx / PT) >> 1);
  }
  static constexpr int rr(int idx) { return 8 * ((idx & 7) >> 2) + (idx & 3); }
  static constexpr int rc_in(int idx) {
    return R == 16 ? rr(idx) : 2 * rr(idx) + (idx % PT) / 8;
  }
  static constexpr int rc_out(int idx) {
    return R == 16 ? rr(idx) : rr(idx) + 16 * ((idx % PT) / 8);
  }
};

// kMfScale F x for 32 columns of exact halves, small terms first.
__device__ __forceinline__ float16v mf_mul(const MfMat& F, const half8v* x) {
  float16v acc = {};
#pragma unroll
  for (int i = kMfParts - 1; i >= 0; --i)
#pragma unroll
    for (int s = 0; s < 2; ++s)
      acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(F.part[i][s], x[s], acc, 0, 0, 0);
  return acc;
}

// A sample's two bytes as halves: 0x6400 | u is the half 1024 + u, so
// byte ^ 0x80 in the mantissa less 1152 is the signed byte, exactly.
__device__ __forceinline__ half2v mf_sample(unsigned w) {
  const unsigned p = __builtin_amdgcn_perm(0x64646464u, w ^ 0x8080u, 0x04010400u);
  const half2v bias = {(_Float16)-1152.0f, (_Float16)-1152.0f};
  return __builtin_bit_cast(half2v, p) + bias;
}

// The first pass, times kMfScale: w[idx] holds the bytes of this thread's sample idx.
template <class S, int R>
__device__ __forceinline__ void mf_first(float2* v, const unsigned* w, const float2* mf, int t) {
  constexpr int PT = R / 2, TILES = S::E / PT;
  const MfMat F = mf_matrix(mf, kMfPlain, t & 63);
  MfMat O;
  if constexpr (R == 32) O = mf_matrix(mf, kMfOdd, t & 63);
#pragma unroll
  for (int q = 0; q < TILES; ++q) {
    float16v y[2];
#pragma unroll
    for (int g = 0; g < PT / 8; ++g) {
      half8v x[2];
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const half2v s = mf_sample(w[q * PT + 8 * g + i]);
        x[i >> 2][2 * (i & 3)] = s[0];
        x[i >> 2][2 * (i & 3) + 1] = s[1];
      }
      y[g] = mf_mul(g ? O : F, x);
    }
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const float2 a = make_float2(y[0][2 * i], y[0][2 * i + 1]);
      if constexpr (R == 16) {
        v[q * 8 + i] = a;
      } else {
        const float2 b = make_float2(y[1][2 * i], y[1][2 * i + 1]);
        v[q * 16 + i] = cadd(a, b);
        v[q * 16 + 8 + i] = csub(a, b);
      }
    }
  }
}

// Outputs of the first pass (column j's points at R j + r) to the inputs of
// the second (radix RN) through LDS, as exchange.
template <class S, int R, int RN>
__device__ __forceinline__ void mf_exchange(float2* v, float* lds, int t) {
  using W = MfMap<S, R>;
  constexpr int E = S::E, T = S::T, NR = S::N / RN;
  const int wp = W::thread_col(t) * R + W::thread_r_out(t);
  auto woff = [](int i) constexpr { return W::cc(i) * R + W::rc_out(i); };
  auto roff = [](int i) constexpr { return T * (i / RN) + (i % RN) * NR; };
  if constexpr (!S::SPLIT) {
    float2* l2 = (float2*)lds;
    const int wb = lpad(wp), rb = lpad(t);
    __syncthreads();
#pragma unroll
    for (int i = 0; i < E; ++i) l2[wb + loff(woff(i))] = v[i];
    __syncthreads();
#pragma unroll
    for (int i = 0; i < E; ++i) v[i] = l2[rb + loff(roff(i))];
  } else {
    constexpr int TS = xpad_shift(R, 1);
    const int wb = xpad<TS>(wp), rb = xpad<TS>(t);
    __syncthreads();
#pragma unroll
    for (int i = 0; i < E; ++i) lds[wb + xpad<TS>(woff(i))] = v[i].x;
    __syncthreads();
    float re[E];
#pragma unroll
    for (int i = 0; i < E; ++i) re[i] = lds[rb + xpad<TS>(roff(i))];
    __syncthreads();
#pragma unroll
    for (int i = 0; i < E; ++i) lds[wb + xpad<TS>(woff(i))] = v[i].y;
    __syncthreads();
#pragma unroll
    for (int i = 0; i < E; ++i) v[i] = make_float2(re[i], lds[rb + xpad<TS>(roff(i))]);
  }
}

// The forward transform from pass 1 on (pass 0 is mf_first).
template <class S>
__device__ __forceinline__ void mf_forward_rest(float2* v, float* lds,
                                                const float2* __restrict__ tw, int t) {
  sfor<1, S::NP>([&](auto P) {
    constexpr int p = decltype(P)::value;
    PassTw<S, S::rad_f(p), S::ns_f(p), S::tw_f(p)> pt;
    if constexpr (S::PF) pt.load(tw, t);
    if constexpr (p == 1)
      mf_exchange<S, S::rad_f(0), S::rad_f(1)>(v, lds, t);
    else
      exchange<S, S::rad_f(p - 1), S::ns_f(p - 1), S::rad_f(p)>(v, lds, t);
    if constexpr (!S::PF) pt.load(tw, t);
    butterflies<S, S::rad_f(p), S::ns_f(p), -1, S::tw_f(p)>(v, pt);
  });
}

}  // namespace cdd
