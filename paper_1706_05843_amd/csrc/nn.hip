// Kernels of the gauge-covariant parallel-transport network (flexible
// preconditioner) and of flexible CG. Not part of the paper's method: the
// layer form, losses and optimiser are this library's choices.
//
// Layer C_in -> C_out, output parity p, 20 terms per channel pair:
//   y_c(x, s) = sum_t sum_c' W[t][c][c'] (S_t X_c')(x, s),
//   S_0 = P_+, S_1 = P_-, S_{2+e} = T_e, S_{10+e} = g_mu(e) T_e (e = 0..7),
//   S_18 X(s) = P_+ X(s-1), S_19 X(s) = P_- X(s+1) (cyclic in s),
// with the eight transports T_e of the hop kernels' per-parity links
// (e < 4: U_mu(x) X(x+mu), mu = e; e >= 4: U_mu(x-mu)^dag X(x-mu), mu = e-4;
// boundary phases included). Activations are packed FP32 half-fields with
// the channel as the right-hand-side index. Weights: bfloat16 pairs
// (re, im) [20][C_out][C_in], FP32 arithmetic.
// Adjoint in X: conj(W[t'][c'][c]) S_t'^dag with T_e^dag = T_{e^4}, g_mu
// Hermitian and commuting with the transports, P_+- Hermitian and the s
// shifts reversed.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "device_common.h"
#include "internal.h"
#include "nn_internal.h"

namespace eofa {

__device__ __forceinline__ float bf16_to_f32(unsigned short b) { return __uint_as_float((unsigned)b << 16); }

__device__ __forceinline__ unsigned short f32_to_bf16(float f) {  // round to nearest even
  unsigned u = __float_as_uint(f);
  u += 0x7FFFu + ((u >> 16) & 1u);
  return (unsigned short)(u >> 16);
}

// z <- L z for a 12-component spinor (colour matvec per spin), L = 9 complex
__device__ __forceinline__ void link_mul(const float2* L, cx<float>* z) {
  cx<float> U[9];
#pragma unroll
  for (int k = 0; k < 9; ++k) U[k] = {L[k].x, L[k].y};
#pragma unroll
  for (int sp = 0; sp < 4; ++sp) {
    const cx<float> a = z[sp * 3], b = z[sp * 3 + 1], c = z[sp * 3 + 2];
#pragma unroll
    for (int r = 0; r < 3; ++r) z[sp * 3 + r] = cfma(U[r * 3 + 2], c, cfma(U[r * 3 + 1], b, cmul(U[r * 3], a)));
  }
}

__device__ __forceinline__ cx<float> times_i(cx<float> a) { return {-a.i, a.r}; }

// one chirality half of a packed FP32 spinor: h = 0 the P_+ components
// 0..5 (into v[0..5]), h = 1 the P_- components 6..11 (into v[6..11])
__device__ __forceinline__ void ld_half32(const float* base, const FD& f, int r, int s, int i, int h,
                                          cx<float>* v) {
  const size_t e0 = eidx(f, r, 0, s, i), qs = qstride(f);
#pragma unroll
  for (int q = 0; q < 3; ++q) ld_pair<P32>(base, e0 + (3 * h + q) * qs, v[6 * h + 2 * q], v[6 * h + 2 * q + 1]);
}

// g = g_mu v in the chiral basis of the field layout:
// g_mu = [[0, A_mu], [A_mu^dag, 0]], A = -i sigma_1, -i sigma_2, -i sigma_3, 1
__device__ __forceinline__ void gamma_mul(int mu, const cx<float>* v, cx<float>* g) {
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    const cx<float> u0 = v[c], u1 = v[3 + c], l0 = v[6 + c], l1 = v[9 + c];
    if (mu == 0) {
      g[c] = -1.f * times_i(l1);
      g[3 + c] = -1.f * times_i(l0);
      g[6 + c] = times_i(u1);
      g[9 + c] = times_i(u0);
    } else if (mu == 1) {
      g[c] = -1.f * l1;
      g[3 + c] = l0;
      g[6 + c] = u1;
      g[9 + c] = -1.f * u0;
    } else if (mu == 2) {
      g[c] = -1.f * times_i(l0);
      g[3 + c] = times_i(l1);
      g[6 + c] = times_i(u0);
      g[9 + c] = -1.f * times_i(u1);
    } else {
      g[c] = l0;
      g[3 + c] = l1;
      g[6 + c] = u0;
      g[9 + c] = u1;
    }
  }
}

// weight of term t from input channel ci to output channel c of this
// application; the adjoint reads conj(W[t][ci][c]) of the forward layer
// (whose C_out is this application's C_in)
template <bool ADJ>
__device__ __forceinline__ cx<float> wload(const NetLayerArgs& a, int t, int c, int ci) {
  const size_t k = ADJ ? (((size_t)t * a.Cin + ci) * a.Cout + c) * 2 : (((size_t)t * a.Cout + c) * a.Cin + ci) * 2;
  const float wr = bf16_to_f32(a.w[k]), wi = bf16_to_f32(a.w[k + 1]);
  return {wr, ADJ ? -wi : wi};
}

// One thread: one 5D site (i, s) of the output parity and a block of CB
// output channels c0 .. c0+CB-1. The work-group first stages the weights it
// needs, W[t][c0+cc][ci] as FP32 complex (conjugated and transposed for the
// adjoint), in LDS: every lane reads the same weight, which LDS broadcasts.
// Per transport direction e the term pair W[2+e] + W[10+e] g_mu is applied
// in one of two orders (g_mu commutes with the link):
//  * TF (transport first): each input channel is transported once and then
//    mixed into the CB outputs: C_in link products, accumulators only;
//  * otherwise mix first: z_c = sum_c' (W[2+e] + W[10+e] g_mu) X_c'(neighbour)
//    for the CB outputs, then one link product per output: CB link products,
//    but CB more spinors of registers.
// Used for the smallest layers (see launch_pt_layer): TF for two to four
// outputs, mix first for one. Registers: 48 CB (accumulators), plus 48 CB for
// mix first.
template <bool ADJ, int CB, bool TF>
__global__ void __launch_bounds__(256) pt_layer_kernel(NetLayerArgs a) {
  __shared__ float2 s_w[NET_TERMS * 4 * NET_MAXC];  // [t][cc][ci], CB <= 4
  const int c0 = blockIdx.y * CB;
  const int nco = min(CB, a.Cout - c0);
  for (int k = threadIdx.x; k < NET_TERMS * CB * a.Cin; k += blockDim.x) {
    const int ci = k % a.Cin, cc = (k / a.Cin) % CB, t = k / (a.Cin * CB);
    float2 w = {0.f, 0.f};
    if (cc < nco) {
      const cx<float> v = wload<ADJ>(a, t, c0 + cc, ci);
      w = {v.r, v.i};
    }
    s_w[k] = w;
  }
  __syncthreads();
  const int idx = blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= a.Vh * a.Ls) return;
  auto W = [&](int t, int cc, int ci) {
    const float2 w = s_w[(t * CB + cc) * a.Cin + ci];
    return cx<float>{w.x, w.y};
  };
  const int i = idx / a.Ls, s = idx - i * a.Ls;
  const int p = a.parity;
  const FD fin = {a.Ls, a.Vh, a.Cin};
  cx<float> acc[CB][12];
#pragma unroll
  for (int cc = 0; cc < CB; ++cc)
#pragma unroll
    for (int k = 0; k < 12; ++k) acc[cc][k] = {0.f, 0.f};
  // same-parity terms: P_+ and P_- at (x, s); P_+ X(s-1) and P_- X(s+1),
  // in the adjoint P_+ X(s+1) and P_- X(s-1)
  {
    const int sm = s == 0 ? a.Ls - 1 : s - 1, sp = s == a.Ls - 1 ? 0 : s + 1;
    const int s_up = ADJ ? sp : sm, s_lo = ADJ ? sm : sp;
    for (int ci = 0; ci < a.Cin; ++ci) {
      cx<float> v[12], xu[12], xl[12];
      ld_spinor<P32>(a.xin[p], fin, ci, s, i, v);
      ld_half32(a.xin[p], fin, ci, s_up, i, 0, xu);
      ld_half32(a.xin[p], fin, ci, s_lo, i, 1, xl);
#pragma unroll
      for (int cc = 0; cc < CB; ++cc) {
        const cx<float> w0 = W(0, cc, ci), w1 = W(1, cc, ci), w18 = W(18, cc, ci), w19 = W(19, cc, ci);
#pragma unroll
        for (int q = 0; q < 6; ++q) acc[cc][q] = cfma(w18, xu[q], cfma(w0, v[q], acc[cc][q]));
#pragma unroll
        for (int q = 6; q < 12; ++q) acc[cc][q] = cfma(w19, xl[q], cfma(w1, v[q], acc[cc][q]));
      }
    }
  }
  for (int e = 0; e < 8; ++e) {
    const int j = a.nbr[(size_t)i * 8 + e];
    const int te = ADJ ? (e ^ 4) : e;  // T_e^dag = T_{e^4}
    const int mu = e & 3;
    const float2* L = (const float2*)a.links + ((size_t)i * 8 + e) * 9;
    if constexpr (TF) {
      for (int ci = 0; ci < a.Cin; ++ci) {
        cx<float> v[12], gv[12];
        ld_spinor<P32>(a.xin[1 - p], fin, ci, s, j, v);
        link_mul(L, v);
        gamma_mul(mu, v, gv);
#pragma unroll
        for (int cc = 0; cc < CB; ++cc) {
          const cx<float> wa = W(2 + te, cc, ci), wb = W(10 + te, cc, ci);
#pragma unroll
          for (int q = 0; q < 12; ++q) acc[cc][q] = cfma(wb, gv[q], cfma(wa, v[q], acc[cc][q]));
        }
      }
    } else {
      cx<float> z[CB][12];
#pragma unroll
      for (int cc = 0; cc < CB; ++cc)
#pragma unroll
        for (int k = 0; k < 12; ++k) z[cc][k] = {0.f, 0.f};
      for (int ci = 0; ci < a.Cin; ++ci) {
        cx<float> v[12], gv[12];
        ld_spinor<P32>(a.xin[1 - p], fin, ci, s, j, v);
        gamma_mul(mu, v, gv);
#pragma unroll
        for (int cc = 0; cc < CB; ++cc) {
          const cx<float> wa = W(2 + te, cc, ci), wb = W(10 + te, cc, ci);
#pragma unroll
          for (int q = 0; q < 12; ++q) z[cc][q] = cfma(wb, gv[q], cfma(wa, v[q], z[cc][q]));
        }
      }
#pragma unroll
      for (int cc = 0; cc < CB; ++cc) {
        if (cc >= nco) break;
        link_mul(L, z[cc]);
#pragma unroll
        for (int q = 0; q < 12; ++q) acc[cc][q] = acc[cc][q] + z[cc][q];
      }
    }
  }
  const FD fo = {a.Ls, a.Vh, a.Cout};
#pragma unroll
  for (int cc = 0; cc < CB; ++cc) {
    if (cc >= nco) break;
    st_spinor<P32>(a.yout, fo, c0 + cc, s, i, acc[cc]);
  }
}

// The layer on the matrix cores. A wave owns 16 consecutive 5D sites (columns
// n = lane % 16) and its four lane groups g = lane / 16 take four transport
// directions at once: in a pass, a lane loads and transports two input channels
// of its column along its group's direction, and one K = 32 MFMA sums over the
// four directions and two channels. With the spins paired by g_mu,
// (g_mu v)_A = k_A v_B and (g_mu v)_B = k_B v_A, k a sign or +-i, the terms of
// a direction on a pair (A, B) are
//   y_A += Wa v_A + k_A Wb v_B,   y_B += k_B Wb v_A + Wa v_B,
// real products of the weights (rows: Re, Im of each output channel; k folded
// in) with (Re v_A, Im v_A, Re v_B, Im v_B) of the channels. A pass takes the
// directions of mu = 0, 1 (pairs (0, 3), (1, 2)) or of mu = 2, 3 (pairs (0, 2),
// (1, 3)), both signs, so that its pairs agree over the wave. A lane ends with
// NCO output channels of its column; nothing moves between lanes by hand.
// The weights are bfloat16 already; an FP32 activation is split exactly into
// three bfloat16 numbers (8 + 8 + 8 bits, each the truncated rest of the one
// before), so the products are those of the FP32 form, summed in FP32. Each pass
// sums into zeros, smallest parts first, and joins the accumulator by a vector
// add: added to a large accumulator inside the MFMA the sums round worse. The
// error of a whole network against 64 bits, FP32 multiply-adds / MFMA into the
// accumulator / as here: 1,8,8,8,1 at 16^3 x 32 x 16 3.7e-7 / 5.9e-7 / 2.5e-7,
// 1,4,1 2.1e-7 / 2.8e-7 / 1.7e-7, 1,3,2,1 at 8^4 x 8 3.6e-7 / 2.8e-7 / 2.1e-7.
// Two things the split does not carry: an infinite activation becomes NaN (in every
// row of its products), and the matrix cores take a part below 2^-126 as zero, so that
// activations below 2^-102 lose digits. A lane whose sums hold a NaN or lie below
// MF_TINY (2^12 above that line) does its outputs over as plain FP32 products (mf_plain).
// What bounds it: vector instructions (6000 per wave and tile of 16 5D sites at 8 -> 8
// channels: transports 288 and splits 264 of each pass), busy four fifths of the
// time, and the 5.3 GB a launch that miss the L2 (5.5 TB/s); the matrix cores are busy
// 17 %. Taking two channels of all directions per pass instead of one direction of
// all channels keeps the columns the XCD's tiles gather at one time within its 4 MB
// L2 (with 8 channels at once 69 % of the L2 requests missed, 6.4 GB a launch): 8 -> 8
// channels, 16^3 x 32 x 16, 1169 -> 985 us, with the outputs streamed past the MALL
// 948 us (and 2.5 % for the accuracy of the sums); one thread per site, two outputs
// at a time, took 4067 us.
typedef __bf16 b8_t __attribute__((ext_vector_type(8)));
typedef float f32x4_t __attribute__((ext_vector_type(4)));
typedef unsigned w4_t __attribute__((ext_vector_type(4)));

constexpr int MF_MAXP = (NET_MAXC + 1) / 2;      // channel pairs
constexpr int MF_FRAGS = MF_MAXP * 8 + 2;        // [pair of channels][mu class][spin pair][output], same-site upper, lower
constexpr int MF_SITES = 9;                      // most 4D sites 16 consecutive 5D sites touch (Ls >= 2)
constexpr int MF_LSTR = 73;                      // link stride in LDS
constexpr float MF_TINY = 0x1p-90f;              // largest sum that is looked at again

__device__ __forceinline__ f32x4_t mf_mul(w4_t A, w4_t B, f32x4_t c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(b8_t, A), __builtin_bit_cast(b8_t, B), c, 0, 0, 0);
}

// the three bfloat16 parts of a complex number as (Re, Im) words
__device__ __forceinline__ void mf_split(cx<float> v, unsigned& hi, unsigned& mid, unsigned& lo) {
  const unsigned r = __float_as_uint(v.r), i = __float_as_uint(v.i);
  hi = __builtin_amdgcn_perm(i, r, 0x07060302u);
  const float r1 = v.r - __uint_as_float(r & 0xFFFF0000u), i1 = v.i - __uint_as_float(i & 0xFFFF0000u);
  const unsigned ur = __float_as_uint(r1), ui = __float_as_uint(i1);
  mid = __builtin_amdgcn_perm(ui, ur, 0x07060302u);
  const float r2 = r1 - __uint_as_float(ur & 0xFFFF0000u), i2 = i1 - __uint_as_float(ui & 0xFFFF0000u);
  lo = __builtin_amdgcn_perm(__float_as_uint(i2), __float_as_uint(r2), 0x07060302u);
}

// direction of lane group g in a pass of mu class h
__device__ __forceinline__ int mf_dir(int h, int g) { return 2 * h + (g & 1) + 4 * (g >> 1); }

// weight W[t][co][ci] (conjugated and transposed in the adjoint) times i^rot,
// as bfloat16 bits (Re, Im)
template <bool ADJ>
__device__ __forceinline__ uint2 mf_weight(const NetLayerArgs& a, int t, int rot, int co, int ci) {
  const size_t k = ADJ ? (((size_t)t * a.Cin + ci) * a.Cout + co) * 2 : (((size_t)t * a.Cout + co) * a.Cin + ci) * 2;
  unsigned r = a.w[k], i = a.w[k + 1];
  if (ADJ) i ^= 0x8000u;
  if (rot & 1) {  // i w = (-Im, Re)
    const unsigned x = r;
    r = i ^ 0x8000u;
    i = x;
  }
  if (rot & 2) {
    r ^= 0x8000u;
    i ^= 0x8000u;
  }
  return make_uint2(r, i);
}

// lane (row, g)'s eight K values of fragment f: word h holds the row's factors
// of (Re, Im) of operand word h (channel h / 2 of the pair, spin A or B by h % 2)
template <bool ADJ, int NCO>
__device__ __forceinline__ w4_t mf_fragment(const NetLayerArgs& a, int f, int row, int g) {
  const int co = NCO == 2 ? row >> 1 : row >> 2, ri = NCO == 2 ? row & 1 : row & 3;
  w4_t w;
#pragma unroll
  for (int h = 0; h < 4; ++h) {
    const int part = h & 1;
    int ci, t, rot = 0;
    if (f >= MF_MAXP * 8) {  // same-site terms: group g holds channels 2g, 2g + 1
      const int lower = f - MF_MAXP * 8;
      ci = 2 * g + (h >> 1);
      t = part ? 18 + lower : lower;
    } else {
      const int cls = (f >> 2) & 1, pair = (f >> 1) & 1, low = f & 1;
      const int e = mf_dir(cls, g), mu = e & 3, te = ADJ ? (e ^ 4) : e;  // T_e^dag = T_{e^4}
      ci = 2 * (f >> 3) + (h >> 1);
      t = part == low ? 2 + te : 10 + te;
      if (part != low) {  // k of (mu, pair, output): -i = i^3, -1 = i^2
        if (mu == 0)
          rot = low ? 1 : 3;
        else if (mu == 1)
          rot = pair ? 0 : 2;
        else if (mu == 2)
          rot = (low != pair) ? 1 : 3;
      }
    }
    unsigned v = 0;
    if (co < a.Cout && ci < a.Cin && ri < 2) {
      const uint2 z = mf_weight<ADJ>(a, t, rot, co, ci);
      v = ri == 0 ? (z.x | ((z.y ^ 0x8000u) << 16)) : (z.y | (z.x << 16));
    }
    w[h] = v;
  }
  return w;
}

struct MfIn {
  cx<float> v[2][12];  // two channels
};
// channels c0, c0 + 1 at the 5D site of byte offset off within a plane; a
// channel past the last reads the last one again (its weights are zero)
__device__ __forceinline__ void mf_load(const float* base, const FD& f, int c0, unsigned off, MfIn& x) {
#pragma unroll
  for (int ch = 0; ch < 2; ++ch) {
    const char* plane = (const char*)base + (size_t)min(c0 + ch, f.nrhs - 1) * 6 * qstride(f) * 16;
#pragma unroll
    for (int q = 0; q < 6; ++q) {
      const float4 v = *(const float4*)(plane + q * qstride(f) * 16 + off);
      x.v[ch][2 * q] = {v.x, v.y};
      x.v[ch][2 * q + 1] = {v.z, v.w};
    }
  }
}

// the split operand words of one spin pair and colour: (A, B) of both channels
__device__ __forceinline__ void mf_operand(const cx<float>* va, const cx<float>* vb, w4_t* B) {
#pragma unroll
  for (int ch = 0; ch < 2; ++ch) {
    unsigned h, m, l;
    mf_split(va[ch], h, m, l);
    B[0][2 * ch] = h;
    B[1][2 * ch] = m;
    B[2][2 * ch] = l;
    mf_split(vb[ch], h, m, l);
    B[0][2 * ch + 1] = h;
    B[1][2 * ch + 1] = m;
    B[2][2 * ch + 1] = l;
  }
}

// one pass: transport the loaded channels along this lane's direction and
// accumulate both outputs of each spin pair; LO: mu = 0, 1
template <bool LO>
__device__ __forceinline__ void mf_pass(const MfIn& x, const float2* L, const w4_t* frag, f32x4_t* acc) {
  cx<float> U[9];
#pragma unroll
  for (int k = 0; k < 9; ++k) U[k] = {L[k].x, L[k].y};
#pragma unroll
  for (int pair = 0; pair < 2; ++pair) {
    const int sa = pair, sb = LO ? 3 - pair : 2 + pair;
    const w4_t M1 = frag[(pair * 2) * 64], M2 = frag[(pair * 2 + 1) * 64];
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      cx<float> va[2], vb[2];
#pragma unroll
      for (int ch = 0; ch < 2; ++ch) {
        const cx<float>* p = x.v[ch] + sa * 3;
        const cx<float>* q = x.v[ch] + sb * 3;
        va[ch] = cfma(U[c * 3 + 2], p[2], cfma(U[c * 3 + 1], p[1], cmul(U[c * 3], p[0])));
        vb[ch] = cfma(U[c * 3 + 2], q[2], cfma(U[c * 3 + 1], q[1], cmul(U[c * 3], q[0])));
      }
      w4_t B[3];
      mf_operand(va, vb, B);
      f32x4_t ya = {0.f, 0.f, 0.f, 0.f}, yb = ya;
#pragma unroll
      for (int k = 2; k >= 0; --k) {
        ya = mf_mul(M1, B[k], ya);
        yb = mf_mul(M2, B[k], yb);
      }
      acc[sa * 3 + c] += ya;
      acc[sb * 3 + c] += yb;
    }
  }
}

// Output channels c0 .. c0 + nc - 1 of one 5D site as plain FP32 products, for the
// few sites whose operands the split does not carry. Rolled up: its speed does not
// matter, its registers must not weigh on the kernel around it.
template <bool ADJ>
__device__ __forceinline__ void mf_plain(const NetLayerArgs& a, int k5, int s, int c0, int nc) {
  const int i = a.order[k5], Ls = a.Ls, p = a.parity;
  const FD fin = {Ls, a.Vh, a.Cin}, fo = {Ls, a.Vh, a.Cout};
  const int sm = s == 0 ? Ls - 1 : s - 1, sp = s == Ls - 1 ? 0 : s + 1;
#pragma unroll 1
  for (int co = c0; co < min(c0 + nc, a.Cout); ++co) {
    cx<float> y[12];
#pragma unroll
    for (int k = 0; k < 12; ++k) y[k] = {0.f, 0.f};
#pragma unroll 1
    for (int ci = 0; ci < a.Cin; ++ci) {
      cx<float> v[12], w[12];
      ld_spinor<P32>(a.xin[p], fin, ci, s, i, v);
      ld_half32(a.xin[p], fin, ci, ADJ ? sp : sm, i, 0, w);
      ld_half32(a.xin[p], fin, ci, ADJ ? sm : sp, i, 1, w);
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const cx<float> wv = wload<ADJ>(a, h, co, ci), ww = wload<ADJ>(a, 18 + h, co, ci);
#pragma unroll
        for (int k = 6 * h; k < 6 * h + 6; ++k) y[k] = cfma(ww, w[k], cfma(wv, v[k], y[k]));
      }
#pragma unroll 1
      for (int e = 0; e < 8; ++e) {
        ld_spinor<P32>(a.xin[1 - p], fin, ci, s, a.nbr[(size_t)i * 8 + e], v);
        link_mul((const float2*)a.links + ((size_t)i * 8 + e) * 9, v);
        gamma_mul(e & 3, v, w);
        const int te = ADJ ? (e ^ 4) : e;  // T_e^dag = T_{e^4}
        const cx<float> wv = wload<ADJ>(a, 2 + te, co, ci), ww = wload<ADJ>(a, 10 + te, co, ci);
#pragma unroll
        for (int k = 0; k < 12; ++k) y[k] = cfma(ww, w[k], cfma(wv, v[k], y[k]));
      }
    }
    st_spinor<P32>(a.yout, fo, co, s, i, y);
  }
}

template <bool ADJ, int NCO>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 8))) pt_mfma_kernel(NetLayerArgs a, bool nt) {
  extern __shared__ w4_t s_frag[];  // [npair * 8 + 2][64]
  __shared__ float2 s_link[4 * MF_SITES * MF_LSTR];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), n = lane & 15, g = lane >> 4;
  const int npair = (a.Cin + 1) / 2;
  for (int j = tid; j < (npair * 8 + 2) * 64; j += 256) {
    const int f = j >> 6;
    s_frag[j] = mf_fragment<ADJ, NCO>(a, f < npair * 8 ? f : MF_MAXP * 8 + f - npair * 8, j & 15, (j >> 4) & 3);
  }
  __syncthreads();
  const int n5 = a.Vh * a.Ls, Ls = a.Ls, p = a.parity;
  const int ntile = (n5 + 63) / 64;
  const FD fin = {Ls, a.Vh, a.Cin}, fo = {Ls, a.Vh, a.Cout};
  const w4_t* frag = s_frag + lane;
  const float* xo = a.xin[1 - p];
  float2* wl = s_link + wave * MF_SITES * MF_LSTR;
  const int e0 = mf_dir(0, g), e1 = mf_dir(1, g);
  MfIn x0, x1;
  // each XCD a contiguous run of tiles (work-groups are dealt round-robin; with
  // fewer than 8 work-groups, each its own run)
  const int nrun = min(8, (int)gridDim.x), run = blockIdx.x % nrun, nx = ((int)gridDim.x + nrun - 1 - run) / nrun;
  const int t0 = (int)((size_t)ntile * run / nrun), t1 = (int)((size_t)ntile * (run + 1) / nrun);
  for (int tile = t0 + (int)blockIdx.x / nrun; tile < t1; tile += nx) {
    const int first = tile * 64 + wave * 16;
    if (first >= n5) continue;  // uniform over the wave; no barrier below
    const int idx = min(first + n, n5 - 1);
    const bool live = first + n < n5;
    const int k5 = idx / Ls, s = idx - k5 * Ls;
    const int i = a.order[k5];
    const int i0 = first / Ls, ns = min(first + 15, n5 - 1) / Ls - i0 + 1;
    __builtin_amdgcn_wave_barrier();
    for (int k = lane; k < ns * 72; k += 64) {
      const int site = k / 72, r = k - site * 72;
      wl[site * MF_LSTR + r] = ((const float2*)a.links)[(size_t)a.order[i0 + site] * 72 + r];
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    const float2* L = wl + (k5 - i0) * MF_LSTR;
    const unsigned nb0 = (unsigned)(a.nbr[(size_t)i * 8 + e0] * Ls + s) * 16u;
    const unsigned nb1 = (unsigned)(a.nbr[(size_t)i * 8 + e1] * Ls + s) * 16u;
    f32x4_t acc[12];
#pragma unroll
    for (int k = 0; k < 12; ++k) acc[k] = {0.f, 0.f, 0.f, 0.f};
    // same-site terms, group g channels 2g and 2g + 1: operand (v, its s
    // neighbour of the same chirality)
    {
      const int sm = s == 0 ? Ls - 1 : s - 1, sp = s == Ls - 1 ? 0 : s + 1;
      const int c0 = min(2 * g, a.Cin - 1), c1 = min(2 * g + 1, a.Cin - 1);
#pragma unroll
      for (int ch = 0; ch < 2; ++ch) {
        ld_spinor<P32>(a.xin[p], fin, ch ? c1 : c0, s, i, x0.v[ch]);
        ld_half32(a.xin[p], fin, ch ? c1 : c0, ADJ ? sp : sm, i, 0, x1.v[ch]);
        ld_half32(a.xin[p], fin, ch ? c1 : c0, ADJ ? sm : sp, i, 1, x1.v[ch]);
      }
      const w4_t fu = frag[npair * 8 * 64], fl = frag[(npair * 8 + 1) * 64];
#pragma unroll
      for (int k = 0; k < 12; ++k) {
        const cx<float> va[2] = {x0.v[0][k], x0.v[1][k]}, vb[2] = {x1.v[0][k], x1.v[1][k]};
        w4_t B[3];
        mf_operand(va, vb, B);
#pragma unroll
        for (int q = 2; q >= 0; --q) acc[k] = mf_mul(k < 6 ? fu : fl, B[q], acc[k]);
      }
    }
    // two channels at a time, both mu classes: the next pass's loads are in flight
    mf_load(xo, fin, 0, nb0, x0);
    for (int cp = 0; cp < npair; ++cp) {
      mf_load(xo, fin, 2 * cp, nb1, x1);
      mf_pass<true>(x0, L + e0 * 9, frag + cp * 8 * 64, acc);
      if (cp + 1 < npair) mf_load(xo, fin, 2 * cp + 2, nb0, x0);
      mf_pass<false>(x1, L + e1 * 9, frag + (cp * 8 + 4) * 64, acc);
    }
    if (live) {
#pragma unroll
      for (int ch = 0; ch < NCO; ++ch) {
        if (NCO * g + ch >= a.Cout) break;
        cx<float> y[12];
#pragma unroll
        for (int k = 0; k < 12; ++k) y[k] = {acc[k][2 * ch], acc[k][2 * ch + 1]};
        if (nt)
          st_spinor_nt<P32>(a.yout, fo, NCO * g + ch, s, i, y);
        else
          st_spinor<P32>(a.yout, fo, NCO * g + ch, s, i, y);
      }
      float sum = 0.f, top = 0.f;
#pragma unroll
      for (int k = 0; k < 12; ++k) {
        sum += acc[k][0];
        top = fmaxf(top, fabsf(acc[k][0]));
      }
      if (!isfinite(sum) || (top > 0.f && top < MF_TINY)) {
        int id = tid;
        asm volatile("" : "+v"(id));  // nothing is kept in registers for this
        const int at = tile * 64 + (id >> 6) * 16 + (id & 15);
        mf_plain<ADJ>(a, at / Ls, at % Ls, NCO * ((id >> 4) & 3), NCO);
      }
    }
  }
}

// dL/dW*[t][c][ci] partial sums: sum over sites of G_c(x) . conj((S_t X_ci)(x)).
// A work-group takes a block of CB output and CI input channels (CB CI <= 4),
// one parity and one of two sets of terms: set 0 the transports of mu = 0, 1 with
// the same-site terms, set 1 those of mu = 2, 3 with the s shifts. A thread loads its
// site's G_c once for all terms of the set and each transported input once for
// all its output channels: the loads (G, then the gathers) bound it, 1.7 KB a
// site for 1 -> 4 channels, where a work-group per term pair and two output
// channels read 5.8 KB. Sites run in the traversal order, a contiguous eighth
// per XCD, so that neighbours meet in its L2. 16^3 x 32, Ls = 16: 1 -> 4 channels
// 489 us a launch, 4 -> 1 783, both 1651 before. (Transporting G instead of X
// where there are fewer outputs saves a third of the multiplications of 4 -> 1
// and took 863.)
constexpr int WG_TERMS = 10;  // terms of a set

__device__ __forceinline__ void wg_acc(const cx<float>* g, const cx<float>* v, float* acc, int q0, int q1) {
  float sr = 0.f, si = 0.f;
#pragma unroll
  for (int q = 0; q < 12; ++q) {  // g conj(v)
    if (q < q0 || q >= q1) continue;
    sr = fmaf(g[q].r, v[q].r, fmaf(g[q].i, v[q].i, sr));
    si = fmaf(g[q].i, v[q].r, fmaf(-g[q].r, v[q].i, si));
  }
  acc[0] += sr;
  acc[1] += si;
}

template <int CB, int CI, int SET>
__device__ __forceinline__ void wgrad_set(const NetGradArgs& a, int c0, int ci0, int p, double* dred) {
  constexpr int NT = WG_TERMS;
  const FD fx = {a.Ls, a.Vh, a.Cin}, fg = {a.Ls, a.Vh, a.Cout};
  float acc[CB][CI][NT][2];
#pragma unroll
  for (int cc = 0; cc < CB; ++cc)
#pragma unroll
    for (int k = 0; k < CI; ++k)
#pragma unroll
      for (int t = 0; t < NT; ++t) acc[cc][k][t][0] = acc[cc][k][t][1] = 0.f;
  const int n = a.Vh * a.Ls, nblk = gridDim.x;
  // a contiguous eighth of the sites per XCD (work-groups are dealt round-robin)
  const int nrun = min(8, nblk), run = blockIdx.x % nrun, nx = (nblk + nrun - 1 - run) / nrun;
  const int lo = (int)((size_t)n * run / nrun), hi = (int)((size_t)n * (run + 1) / nrun);
  for (int idx = lo + (blockIdx.x / nrun) * 256 + threadIdx.x; idx < hi; idx += nx * 256) {
    const int k5 = idx / a.Ls, s = idx - k5 * a.Ls, i = a.order[k5];
    cx<float> g[CB][12];
#pragma unroll
    for (int cc = 0; cc < CB; ++cc) ld_spinor<P32>(a.g[p], fg, min(c0 + cc, a.Cout - 1), s, i, g[cc]);
#pragma unroll
    for (int d = 0; d < 4; ++d) {
      const int mu = 2 * SET + (d & 1), e = mu + 4 * (d >> 1);
      const int j = a.nbr[p][(size_t)i * 8 + e];
      const float2* L = (const float2*)a.links[p] + ((size_t)i * 8 + e) * 9;
#pragma unroll
      for (int k = 0; k < CI; ++k) {
        cx<float> v[12], gv[12];
        ld_spinor<P32>(a.x[1 - p], fx, min(ci0 + k, a.Cin - 1), s, j, v);
        link_mul(L, v);
        gamma_mul(mu, v, gv);
#pragma unroll
        for (int cc = 0; cc < CB; ++cc) {
          wg_acc(g[cc], v, acc[cc][k][2 * d], 0, 12);
          wg_acc(g[cc], gv, acc[cc][k][2 * d + 1], 0, 12);
        }
      }
    }
    // set 0 the same-site chirality halves, set 1 those of the s neighbours
    const int sm = s == 0 ? a.Ls - 1 : s - 1, sp = s == a.Ls - 1 ? 0 : s + 1;
#pragma unroll
    for (int k = 0; k < CI; ++k) {
      const int ci = min(ci0 + k, a.Cin - 1);
      cx<float> v[12];
      ld_half32(a.x[p], fx, ci, SET == 0 ? s : sm, i, 0, v);
      ld_half32(a.x[p], fx, ci, SET == 0 ? s : sp, i, 1, v);
#pragma unroll
      for (int cc = 0; cc < CB; ++cc) {
        wg_acc(g[cc], v, acc[cc][k][8], 0, 6);
        wg_acc(g[cc], v, acc[cc][k][9], 6, 12);
      }
    }
  }
  // FP64 sums over the wave, then over the work-group
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  constexpr int NV = CB * CI * NT * 2;
#pragma unroll
  for (int cc = 0; cc < CB; ++cc)
#pragma unroll
    for (int k = 0; k < CI; ++k)
#pragma unroll
      for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          double v = acc[cc][k][t][h];
#pragma unroll
          for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
          if (lane == 0) dred[wv * NV + ((cc * CI + k) * NT + t) * 2 + h] = v;
        }
  __syncthreads();
  for (int k = threadIdx.x; k < NV; k += 256) {
    const int comp = k & 1, t = (k >> 1) % NT, ch = (k >> 1) / NT, ci = ci0 + ch % CI, c = c0 + ch / CI;
    if (ci >= a.Cin || c >= a.Cout) continue;
    double tsum = 0.0;
    for (int w = 0; w < 4; ++w) tsum += dred[w * NV + k];
    // term index: transports 2 + e and 10 + e, then 0, 1 or 18, 19
    const int d = t >> 1, e = 2 * SET + (d & 1) + 4 * (d >> 1);
    const int term = t < 8 ? (t & 1 ? 10 + e : 2 + e) : t - 8 + 18 * SET;
    const int y = term * a.Cin + ci;
    a.partial[((((size_t)y * 2 + p) * a.Cout + c) * gridDim.x + blockIdx.x) * 2 + comp] = tsum;
  }
}

// grid: (blocks, 2 sets x channel blocks, parity)
template <int CB, int CI>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 8))) pt_wgrad_kernel(NetGradArgs a) {
  __shared__ double red[4 * 4 * WG_TERMS * 2];
  const int set = blockIdx.y & 1, blk = blockIdx.y >> 1, nci = (a.Cin + CI - 1) / CI;
  const int c0 = blk / nci * CB, ci0 = blk % nci * CI, p = blockIdx.z;
  if (set == 0)
    wgrad_set<CB, CI, 0>(a, c0, ci0, p, red);
  else
    wgrad_set<CB, CI, 1>(a, c0, ci0, p, red);
}

// gW[t][c][ci] (+)= sum over parity and blocks as (re, im) doubles: one wave per
// value, lanes over the blocks, then across the lanes (a fixed order)
__global__ void __launch_bounds__(256) pt_wgrad_final(const double* partial, int Cin, int Cout, int nblk,
                                                      int accumulate, double* gw) {
  const int k = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;  // over NET_TERMS*Cout*Cin*2
  if (k >= NET_TERMS * Cout * Cin * 2) return;
  const int comp = k & 1, rest = k >> 1;
  const int ci = rest % Cin, c = (rest / Cin) % Cout, t = rest / (Cin * Cout);
  const int y = t * Cin + ci;
  double s = 0.0;
  for (int p = 0; p < 2; ++p)
    for (int b = lane; b < nblk; b += 64) s += partial[((((size_t)y * 2 + p) * Cout + c) * nblk + b) * 2 + comp];
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) s += __shfl_xor(s, off, 64);
  if (lane == 0) gw[k] = accumulate ? gw[k] + s : s;
}

// residual loss: partial sums of <a, r> (re, im) and |a|^2 over one-channel
// FP32 odd half-fields, as [3][nblk]
__global__ void __launch_bounds__(256) net_dot_kernel(int Vh, int Ls, const float* av, const float* rv,
                                                      double* partial) {
  const FD f = {Ls, Vh, 1};
  double cr = 0.0, ci = 0.0, na = 0.0;
  for (int idx = blockIdx.x * blockDim.x + threadIdx.x; idx < Vh * Ls; idx += gridDim.x * blockDim.x) {
    const int i = idx / Ls, s = idx - i * Ls;
    cx<float> x[12], y[12];
    ld_spinor<P32>(av, f, 0, s, i, x);
    ld_spinor<P32>(rv, f, 0, s, i, y);
#pragma unroll
    for (int q = 0; q < 12; ++q) {  // conj(a) r
      cr += (double)x[q].r * y[q].r + (double)x[q].i * y[q].i;
      ci += (double)x[q].r * y[q].i - (double)x[q].i * y[q].r;
      na += (double)x[q].r * x[q].r + (double)x[q].i * x[q].i;
    }
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    cr += __shfl_xor(cr, off, 64);
    ci += __shfl_xor(ci, off, 64);
    na += __shfl_xor(na, off, 64);
  }
  __shared__ double red[4][3];
  if ((threadIdx.x & 63) == 0) {
    red[threadIdx.x >> 6][0] = cr;
    red[threadIdx.x >> 6][1] = ci;
    red[threadIdx.x >> 6][2] = na;
  }
  __syncthreads();
  if (threadIdx.x < 3) {
    double tsum = 0.0;
    for (int w = 0; w < (int)(blockDim.x + 63) / 64; ++w) tsum += red[w][threadIdx.x];
    partial[threadIdx.x * gridDim.x + blockIdx.x] = tsum;
  }
}

// loss = 1 - |c|^2/(|a|^2 |r|^2), c = <a, r>, and the coefficients of
// dL/da* = alpha a + beta r: alpha = |c|^2/(|a|^4 |r|^2), beta = -conj(c)/(|a|^2 |r|^2)
// as coef = (alpha, Re beta, Im beta); a = 0 (or a non-finite sum) gives
// loss 1 and zero coefficients
__global__ void net_resid_coef_kernel(const double* partial, int nblk, const double* rnorm, double* loss,
                                      double* coef) {
  if (threadIdx.x != 0) return;
  double cr = 0.0, ci = 0.0, na = 0.0;
  for (int b = 0; b < nblk; ++b) {
    cr += partial[b];
    ci += partial[nblk + b];
    na += partial[2 * nblk + b];
  }
  const double nr = *rnorm, c2 = cr * cr + ci * ci;
  const double l = 1.0 - c2 / (na * nr);
  if (!(na > 0.0) || !(nr > 0.0) || !isfinite(l)) {
    *loss = 1.0;
    coef[0] = coef[1] = coef[2] = 0.0;
    return;
  }
  *loss = l;
  coef[0] = c2 / (na * na * nr);
  coef[1] = -cr / (na * nr);
  coef[2] = ci / (na * nr);
}

// out = alpha a + beta r (one-channel FP32 odd half-fields)
__global__ void __launch_bounds__(256) net_combine_kernel(int Vh, int Ls, const float* av, const float* rv,
                                                          const double* coef, float* out) {
  const int idx = blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= Vh * Ls) return;
  const int i = idx / Ls, s = idx - i * Ls;
  const FD f = {Ls, Vh, 1};
  const float al = (float)coef[0];
  const cx<float> be = {(float)coef[1], (float)coef[2]};
  cx<float> x[12], y[12];
  ld_spinor<P32>(av, f, 0, s, i, x);
  ld_spinor<P32>(rv, f, 0, s, i, y);
#pragma unroll
  for (int q = 0; q < 12; ++q) x[q] = cfma(be, y[q], al * x[q]);
  st_spinor<P32>(out, f, 0, s, i, x);
}

// loss seed: G = (y - e)/|e|^2 on the odd sites; partial |y - e|^2
__global__ void __launch_bounds__(256) net_loss_kernel(int Vh, int Ls, const float* y, const float* e, float* g,
                                                       const double* enorm, double* partial) {
  const int idx = blockIdx.x * blockDim.x + threadIdx.x;
  double d2 = 0.0;
  if (idx < Vh * Ls) {
    const int i = idx / Ls, s = idx - i * Ls;
    const FD f = {Ls, Vh, 1};
    cx<float> yv[12], ev[12];
    ld_spinor<P32>(y, f, 0, s, i, yv);
    ld_spinor<P32>(e, f, 0, s, i, ev);
    const float inv = (float)(1.0 / *enorm);
#pragma unroll
    for (int q = 0; q < 12; ++q) {
      const cx<float> d = yv[q] - ev[q];
      d2 += (double)d.r * d.r + (double)d.i * d.i;
      yv[q] = inv * d;
    }
    st_spinor<P32>(g, f, 0, s, i, yv);
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) d2 += __shfl_xor(d2, off, 64);
  __shared__ double red[4];
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = d2;
  __syncthreads();
  if (threadIdx.x == 0) {
    double tsum = 0.0;
    for (int w = 0; w < (int)(blockDim.x + 63) / 64; ++w) tsum += red[w];
    partial[blockIdx.x] = tsum;
  }
}

// Adam on FP32 master weights; gradient = 2 dL/dW* / batch for (Re, Im)
__global__ void net_adam_kernel(int n, float* w, float* m, float* v, const double* gw, double scale, float lr,
                                float b1, float b2, float eps, float bc1, float bc2, unsigned short* wb) {
  const int k = blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= n) return;
  const float g = (float)(2.0 * gw[k] * scale);
  const float mk = b1 * m[k] + (1.f - b1) * g;
  const float vk = b2 * v[k] + (1.f - b2) * g * g;
  m[k] = mk;
  v[k] = vk;
  const float wk = w[k] - lr * (mk / bc1) / (sqrtf(vk / bc2) + eps);
  w[k] = wk;
  wb[k] = f32_to_bf16(wk);
}

__global__ void net_to_bf16_kernel(int n, const float* w, unsigned short* wb) {
  const int k = blockIdx.x * blockDim.x + threadIdx.x;
  if (k < n) wb[k] = f32_to_bf16(w[k]);
}

// complex FP64 BLAS on packed half-fields (one right-hand side)
__global__ void __launch_bounds__(256) cdot_kernel(int n, const double2* a, const double2* b, double* partial) {
  double re = 0.0, im = 0.0;
  for (int k = blockIdx.x * blockDim.x + threadIdx.x; k < n; k += gridDim.x * blockDim.x) {
    const double2 x = a[k], y = b[k];  // conj(x) y
    re += x.x * y.x + x.y * y.y;
    im += x.x * y.y - x.y * y.x;
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    re += __shfl_xor(re, off, 64);
    im += __shfl_xor(im, off, 64);
  }
  __shared__ double red[4][2];
  if ((threadIdx.x & 63) == 0) {
    red[threadIdx.x >> 6][0] = re;
    red[threadIdx.x >> 6][1] = im;
  }
  __syncthreads();
  if (threadIdx.x < 2) {
    double tsum = 0.0;
    for (int w = 0; w < (int)(blockDim.x + 63) / 64; ++w) tsum += red[w][threadIdx.x];
    partial[blockIdx.x * 2 + threadIdx.x] = tsum;
  }
}

// sum of nblk (re, im) partials in a fixed order: 128 strided sums per
// component, then a tree (256 threads)
__device__ __forceinline__ void sum_pairs_256(const double* partial, int nblk, double* red) {
  const int c = threadIdx.x & 1;
  double s = 0.0;
  for (int b = threadIdx.x >> 1; b < nblk; b += 128) s += partial[b * 2 + c];
  red[threadIdx.x] = s;
  __syncthreads();
  for (int w = 128; w >= 2; w >>= 1) {  // w even: t and t + w hold the same component
    if ((int)threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
    __syncthreads();
  }
}

__global__ void __launch_bounds__(256) partial_sum2_kernel(const double* partial, int nblk, double* out) {
  __shared__ double red[256];
  sum_pairs_256(partial, nblk, red);
  if (threadIdx.x < 2) out[threadIdx.x] = red[threadIdx.x];
}

// <q_j, z> partial sums for j < nq, as [nq][nblk][2]
__global__ void __launch_bounds__(256) cdot_multi_kernel(int n, int nq, FgPtrs q, const double2* z, double* partial) {
  double re[FG_CHUNK], im[FG_CHUNK];
#pragma unroll
  for (int j = 0; j < FG_CHUNK; ++j) re[j] = im[j] = 0.0;
  for (int k = blockIdx.x * blockDim.x + threadIdx.x; k < n; k += gridDim.x * blockDim.x) {
    const double2 y = z[k];
#pragma unroll
    for (int j = 0; j < FG_CHUNK; ++j) {
      if (j >= nq) break;
      const double2 x = ((const double2*)q.v[j])[k];  // conj(x) y
      re[j] += x.x * y.x + x.y * y.y;
      im[j] += x.x * y.y - x.y * y.x;
    }
  }
  __shared__ double red[4][2 * FG_CHUNK];
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
#pragma unroll
  for (int j = 0; j < FG_CHUNK; ++j) {
    if (j >= nq) break;
    double a = re[j], b = im[j];
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
      a += __shfl_xor(a, off, 64);
      b += __shfl_xor(b, off, 64);
    }
    if (lane == 0) {
      red[wv][2 * j] = a;
      red[wv][2 * j + 1] = b;
    }
  }
  __syncthreads();
  if ((int)threadIdx.x < 2 * nq) {
    double tsum = 0.0;
    for (int w = 0; w < (int)(blockDim.x + 63) / 64; ++w) tsum += red[w][threadIdx.x];
    partial[((size_t)(threadIdx.x >> 1) * gridDim.x + blockIdx.x) * 2 + (threadIdx.x & 1)] = tsum;
  }
}

// work-group j: beta_j = -<q_j, z> / ww_j; bad = 1 if ww_j is not a positive
// finite number or beta_j is not finite
__global__ void __launch_bounds__(256) fgcg_coef_kernel(const double* partial, int nblk, FgPtrs q, double* beta,
                                                        int* bad) {
  const int j = blockIdx.x;
  __shared__ double red[256];
  sum_pairs_256(partial + (size_t)j * nblk * 2, nblk, red);
  if (threadIdx.x != 0) return;
  const double d = *q.ww[j];
  const double re = -red[0] / d, im = -red[1] / d;
  if (!(d > 0.0) || !isfinite(d) || !isfinite(re) || !isfinite(im)) {
    *bad = 1;
    beta[2 * j] = beta[2 * j + 1] = 0.0;
    return;
  }
  beta[2 * j] = re;
  beta[2 * j + 1] = im;
}

// p += sum_j beta_j p_j, j in order
__global__ void __launch_bounds__(256) caxpy_multi_kernel(int n, int nq, FgPtrs pp, const double* beta, double2* p) {
  const int k = blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= n) return;
  double2 acc = p[k];
#pragma unroll
  for (int j = 0; j < FG_CHUNK; ++j) {
    if (j >= nq) break;
    const double br = beta[2 * j], bi = beta[2 * j + 1];
    const double2 a = ((const double2*)pp.v[j])[k];
    acc.x += br * a.x - bi * a.y;
    acc.y += br * a.y + bi * a.x;
  }
  p[k] = acc;
}

// y = y + alpha x  (alpha complex)
__global__ void caxpy_kernel(int n, double ar, double ai, const double2* x, double2* y) {
  const int k = blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= n) return;
  const double2 a = x[k];
  double2 b = y[k];
  b.x += ar * a.x - ai * a.y;
  b.y += ar * a.y + ai * a.x;
  y[k] = b;
}

// p = z + beta p  (beta complex)
__global__ void cxpby_kernel(int n, const double2* z, double br, double bi, double2* p) {
  const int k = blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= n) return;
  const double2 a = p[k], zz = z[k];
  p[k] = make_double2(zz.x + br * a.x - bi * a.y, zz.y + br * a.y + bi * a.x);
}

// e_k = x* - x_k for stored FP32 iterates
__global__ void sub_from_kernel(size_t n, const float* xs, float* e) {
  const size_t k = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (k < n) e[k] = xs[k] - e[k];
}

// out = sign * num / den (num complex, den real); bad = 1 if den is not a
// positive finite number or the quotient is not finite
__global__ void fgcg_ratio_kernel(const double* num, const double* den, double sign, double* out, int* bad) {
  if (threadIdx.x != 0) return;
  const double d = *den;
  const double re = sign * num[0] / d, im = sign * num[1] / d;
  if (!(d > 0.0) || !isfinite(d) || !isfinite(re) || !isfinite(im)) {
    *bad = 1;
    out[0] = out[1] = 0.0;
    return;
  }
  out[0] = re;
  out[1] = im;
}

// p = z + beta p  (beta complex, on the device)
__global__ void cxpby_dev_kernel(int n, const double2* z, const double* beta, double2* p) {
  const int k = blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= n) return;
  const double br = beta[0], bi = beta[1];
  const double2 a = p[k], zz = z[k];
  p[k] = make_double2(zz.x + br * a.x - bi * a.y, zz.y + br * a.y + bi * a.x);
}

// y += alpha x  (alpha complex, on the device)
__global__ void caxpy_dev_kernel(int n, const double* alpha, const double2* x, double2* y) {
  const int k = blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= n) return;
  const double ar = alpha[0], ai = alpha[1];
  const double2 a = x[k];
  double2 b = y[k];
  b.x += ar * a.x - ai * a.y;
  b.y += ar * a.y + ai * a.x;
  y[k] = b;
}

// x += alpha p, r -= alpha q, s -= alpha w; partial |r|^2 and |s|^2 per block
__global__ void __launch_bounds__(256) fgcg_update_kernel(int n, const double* alpha, double2* x, double2* r,
                                                          double2* s, const double2* p, const double2* q,
                                                          const double2* w, double* partial) {
  const double ar = alpha[0], ai = alpha[1];
  double nr = 0.0, ns = 0.0;
  for (int k = blockIdx.x * blockDim.x + threadIdx.x; k < n; k += gridDim.x * blockDim.x) {
    const double2 pk = p[k], qk = q[k], wk = w[k];
    double2 xk = x[k], rk = r[k], sk = s[k];
    xk.x += ar * pk.x - ai * pk.y;
    xk.y += ar * pk.y + ai * pk.x;
    rk.x -= ar * qk.x - ai * qk.y;
    rk.y -= ar * qk.y + ai * qk.x;
    sk.x -= ar * wk.x - ai * wk.y;
    sk.y -= ar * wk.y + ai * wk.x;
    x[k] = xk;
    r[k] = rk;
    s[k] = sk;
    nr += rk.x * rk.x + rk.y * rk.y;
    ns += sk.x * sk.x + sk.y * sk.y;
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    nr += __shfl_xor(nr, off, 64);
    ns += __shfl_xor(ns, off, 64);
  }
  __shared__ double red[4][2];
  if ((threadIdx.x & 63) == 0) {
    red[threadIdx.x >> 6][0] = nr;
    red[threadIdx.x >> 6][1] = ns;
  }
  __syncthreads();
  if (threadIdx.x < 2) {
    double tsum = 0.0;
    for (int wv = 0; wv < (int)(blockDim.x + 63) / 64; ++wv) tsum += red[wv][threadIdx.x];
    partial[threadIdx.x * gridDim.x + blockIdx.x] = tsum;  // [2][nblk]
  }
}

// ---------------------------------------------------------------------------

template <int CB, bool TF>
void launch_pt_layer_cb(const NetLayerArgs& a, bool adj, hipStream_t st) {
  dim3 grid((a.Vh * a.Ls + 255) / 256, (a.Cout + CB - 1) / CB);
  if (adj)
    hipLaunchKernelGGL((pt_layer_kernel<true, CB, TF>), grid, dim3(256), 0, st, a);
  else
    hipLaunchKernelGGL((pt_layer_kernel<false, CB, TF>), grid, dim3(256), 0, st, a);
}

template <int NCO>
void launch_pt_mfma(const NetLayerArgs& a, bool adj, hipStream_t st) {
  const int ntile = (a.Vh * a.Ls + 63) / 64;
  const dim3 grid(std::min(ntile, 512));
  const size_t lds = (size_t)((a.Cin + 1) / 2 * 8 + 2) * 64 * sizeof(w4_t);
  const bool nt = (size_t)96 * a.Vh * a.Ls * (2 * a.Cin + a.Cout) > (size_t(256) << 20);
  if (adj)
    hipLaunchKernelGGL((pt_mfma_kernel<true, NCO>), grid, dim3(256), lds, st, a, nt);
  else
    hipLaunchKernelGGL((pt_mfma_kernel<false, NCO>), grid, dim3(256), lds, st, a, nt);
}

// Which kernel, measured on every channel pair at 16^3 x 32, Ls = 16 (us per
// launch, one thread per site against the matrix cores): 1 -> 4 227 / 323,
// 2 -> 2 277 / 341, 3 -> 1 402 / 455 stay; 1 -> 5 403 / 350, 2 -> 3 359 / 353,
// 3 -> 2 505 / 474, 4 -> 1 538 / 469, 4 -> 4 659 / 532, 8 -> 4 2113 / 885,
// 8 -> 8 4067 / 948 move; the same line holds at 8 x 12 x 6 x 16, Ls = 8
// (4 -> 1 34 / 29, 8 -> 8 104 / 51, 1 -> 4 20 / 20).
// One thread per site: one output channel mixes first (one link product per
// direction), more outputs (of one or two inputs) transport first.
void launch_pt_layer(const NetLayerArgs& a, bool adj, hipStream_t st) {
  if (a.Cin >= 4 || a.Cin * a.Cout >= 5) {
    if (a.Cout > 4)
      launch_pt_mfma<2>(a, adj, st);
    else
      launch_pt_mfma<1>(a, adj, st);
    return;
  }
  if (a.Cout == 1)
    launch_pt_layer_cb<1, false>(a, adj, st);
  else if (a.Cout == 2)
    launch_pt_layer_cb<2, true>(a, adj, st);
  else
    launch_pt_layer_cb<4, true>(a, adj, st);
}

template <int CB, int CI>
void launch_wgrad_cb(const NetGradArgs& a, int nblk, hipStream_t st) {
  const dim3 grid(nblk, 2 * ((a.Cout + CB - 1) / CB) * ((a.Cin + CI - 1) / CI), 2);
  hipLaunchKernelGGL((pt_wgrad_kernel<CB, CI>), grid, dim3(256), 0, st, a);
}

// four outputs of one input per thread, unless there are fewer outputs
void launch_pt_wgrad(const NetGradArgs& a, int nblk, int accumulate, double* gw, hipStream_t st) {
  if (a.Cout == 1)
    launch_wgrad_cb<1, 4>(a, nblk, st);
  else if (a.Cout == 2)
    launch_wgrad_cb<2, 2>(a, nblk, st);
  else
    launch_wgrad_cb<4, 1>(a, nblk, st);
  const int n = NET_TERMS * a.Cout * a.Cin * 2;
  hipLaunchKernelGGL(pt_wgrad_final, dim3((n + 3) / 4), dim3(256), 0, st, a.partial, a.Cin, a.Cout, nblk, accumulate,
                     gw);
}

void launch_net_resid(int Vh, int Ls, const float* av, const float* rv, const double* rnorm, double* partial,
                      double* loss, double* coef, float* out, hipStream_t st) {
  const int n = Vh * Ls;
  const int nblk = std::min(NET_DOT_BLOCKS, (n + 255) / 256);
  hipLaunchKernelGGL(net_dot_kernel, dim3(nblk), dim3(256), 0, st, Vh, Ls, av, rv, partial);
  hipLaunchKernelGGL(net_resid_coef_kernel, dim3(1), dim3(64), 0, st, partial, nblk, rnorm, loss, coef);
  hipLaunchKernelGGL(net_combine_kernel, dim3((n + 255) / 256), dim3(256), 0, st, Vh, Ls, av, rv, coef, out);
}

int launch_net_loss(int Vh, int Ls, const float* y, const float* e, float* g, const double* enorm, double* partial,
                    hipStream_t st) {
  const int nblk = (Vh * Ls + 255) / 256;
  hipLaunchKernelGGL(net_loss_kernel, dim3(nblk), dim3(256), 0, st, Vh, Ls, y, e, g, enorm, partial);
  return nblk;
}

void launch_net_adam(int n, float* w, float* m, float* v, const double* gw, double scale, float lr, float b1,
                     float b2, float eps, int step, unsigned short* wb, hipStream_t st) {
  const float bc1 = 1.f - powf(b1, (float)step), bc2 = 1.f - powf(b2, (float)step);
  hipLaunchKernelGGL(net_adam_kernel, dim3((n + 255) / 256), dim3(256), 0, st, n, w, m, v, gw, scale, lr, b1, b2,
                     eps, bc1, bc2, wb);
}

void launch_net_to_bf16(int n, const float* w, unsigned short* wb, hipStream_t st) {
  hipLaunchKernelGGL(net_to_bf16_kernel, dim3((n + 255) / 256), dim3(256), 0, st, n, w, wb);
}

void launch_cdot(int n, const void* a, const void* b, double* partial, double* out, hipStream_t st) {
  const int nblk = 512;
  hipLaunchKernelGGL(cdot_kernel, dim3(nblk), dim3(256), 0, st, n, (const double2*)a, (const double2*)b, partial);
  hipLaunchKernelGGL(partial_sum2_kernel, dim3(1), dim3(256), 0, st, partial, nblk, out);
}

void launch_fgcg_orth_coefs(int n, int nq, const FgPtrs& q, const void* z, double* partial, double* beta, int* bad,
                            hipStream_t st) {
  const int nblk = 512;
  hipLaunchKernelGGL(cdot_multi_kernel, dim3(nblk), dim3(256), 0, st, n, nq, q, (const double2*)z, partial);
  hipLaunchKernelGGL(fgcg_coef_kernel, dim3(nq), dim3(256), 0, st, partial, nblk, q, beta, bad);
}

void launch_caxpy_multi(int n, int nq, const FgPtrs& pp, const double* beta, void* p, hipStream_t st) {
  hipLaunchKernelGGL(caxpy_multi_kernel, dim3((n + 255) / 256), dim3(256), 0, st, n, nq, pp, beta, (double2*)p);
}

void launch_caxpy(int n, double ar, double ai, const void* x, void* y, hipStream_t st) {
  hipLaunchKernelGGL(caxpy_kernel, dim3((n + 255) / 256), dim3(256), 0, st, n, ar, ai, (const double2*)x,
                     (double2*)y);
}

void launch_cxpby(int n, const void* z, double br, double bi, void* p, hipStream_t st) {
  hipLaunchKernelGGL(cxpby_kernel, dim3((n + 255) / 256), dim3(256), 0, st, n, (const double2*)z, br, bi,
                     (double2*)p);
}

void launch_sub_from(size_t n, const float* xs, float* e, hipStream_t st) {
  hipLaunchKernelGGL(sub_from_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, n, xs, e);
}

void launch_fgcg_ratio(const double* num, const double* den, double sign, double* out, int* bad, hipStream_t st) {
  hipLaunchKernelGGL(fgcg_ratio_kernel, dim3(1), dim3(64), 0, st, num, den, sign, out, bad);
}

void launch_cxpby_dev(int n, const void* z, const double* beta, void* p, hipStream_t st) {
  hipLaunchKernelGGL(cxpby_dev_kernel, dim3((n + 255) / 256), dim3(256), 0, st, n, (const double2*)z, beta,
                     (double2*)p);
}

void launch_caxpy_dev(int n, const double* alpha, const void* x, void* y, hipStream_t st) {
  hipLaunchKernelGGL(caxpy_dev_kernel, dim3((n + 255) / 256), dim3(256), 0, st, n, alpha, (const double2*)x,
                     (double2*)y);
}

int launch_fgcg_update(int n, const double* alpha, void* x, void* r, void* s, const void* p, const void* q,
                       const void* w, double* partial, hipStream_t st) {
  const int nblk = std::min(1024, (n + 255) / 256);
  hipLaunchKernelGGL(fgcg_update_kernel, dim3(nblk), dim3(256), 0, st, n, alpha, (double2*)x, (double2*)r,
                     (double2*)s, (const double2*)p, (const double2*)q, (const double2*)w, partial);
  return nblk;
}

}  // namespace eofa
