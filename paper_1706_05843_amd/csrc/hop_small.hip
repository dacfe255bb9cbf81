// The hop kernel for launches of few waves (see hop_is_small).
//
// On a small lattice the general kernel (kernels.hip: one lane per 5D site) is
// one pass of a few waves over its 10 to 22 KB of straight-line code; most SIMDs
// have nothing to do, and the wave's own instruction stream, about 2000
// instructions at 4 cycles and more, is what the launch waits for (loading all
// eight neighbours at once changed nothing). Here eight waves share the tile of
// one: first each takes one of the eight directions (a gather, the D~ premix, the
// spin projection, one SU(3) product) and leaves its half spinor in LDS; then
// six of them take one component pair each (the pairs q of the packed layout)
// through the sum over the directions, the epilogue along s and the update,
// since M_ee, D~ and their inverses act on every component alike. In FP16S the
// six then meet once more for the site's scale. A CG iteration at 8^4 x 8, one
// system: FP64 65 -> 39 us, FP32 52 -> 30, FP16S 48 -> 29.
#include <hip/hip_runtime.h>

#include "device_common.h"
#include "hop_common.h"
#include "internal.h"

namespace eofa {

namespace {

constexpr int SMW = 8;  // waves per work-group: one per direction

template <class R>
__device__ __forceinline__ cx<R> shfl2(cx<R> v, int src) {
  return {__shfl(v.r, src, 64), __shfl(v.i, src, 64)};
}

// Fifth-dimension neighbours of lane (g, s) for one chirality: L_+ takes s - 1
// (-m across the wrap), L_- takes s + 1; the transposes the other one.
template <class R>
struct SCol {
  int dn, up;    // lanes of s - 1 and s + 1 (cyclic)
  R fdn, fup;    // 1, or -m across the wrap
  bool plus;     // the P_+ half
};

// z += k (L y), or k (L^T y); z may be y
template <class R, bool TRANS>
__device__ __forceinline__ void lacc2(cx<R>* z, const cx<R>* y, const SCol<R>& n, R k) {
  const bool dn = n.plus != TRANS;
  const int src = dn ? n.dn : n.up;
  const R f = (dn ? n.fdn : n.fup) * k;
#pragma unroll
  for (int c = 0; c < 2; ++c) {
    const cx<R> t = shfl2(y[c], src);
    z[c] = cfma_r(f, t, z[c]);
  }
}

// z <- sum_{k<Ls} (x L)^k z (TRANS: L^T), one pass per prime factor of Ls, one
// rounding per term
template <class R, bool TRANS>
__device__ __forceinline__ void series2(cx<R>* z, int s, int g, int Ls, R x, R m, bool plus) {
  const bool dn = plus != TRANS;
  int n = 1, rest = Ls;
  R rn = x;  // x^n
  while (rest > 1) {
    int p = 2;
    while (rest % p != 0) ++p;
    cx<R> sum[2] = {z[0], z[1]};
    R rj = R(1);
    for (int k = 1; k < p; ++k) {
      const int j = k * n;
      rj *= rn;
      const int t = dn ? s - j : s + j;
      const bool wrap = dn ? t < 0 : t >= Ls;
      const int src = g * Ls + (wrap ? (dn ? t + Ls : t - Ls) : t);
      const R f = wrap ? -m * rj : rj;
#pragma unroll
      for (int c = 0; c < 2; ++c) sum[c] = cfma_r(f, shfl2(z[c], src), sum[c]);
    }
#pragma unroll
    for (int c = 0; c < 2; ++c) z[c] = sum[c];
    rn *= rj;
    n *= p;
    rest /= p;
  }
}

// sum over the column of w v, in every lane of it
template <class R>
__device__ __forceinline__ cx<R> col_sum(cx<R> v, int g, int Ls) {
  cx<R> t = {R(0), R(0)};
  for (int q = 0; q < Ls; ++q) t = t + shfl2(v, g * Ls + q);
  return t;
}

// out_s = sum_s' M[s][s'] v_s' of one chirality's dense matrix
template <class R>
__device__ __forceinline__ void dense2(const double* M, const cx<R>* v, cx<R>* out, int s, int g, int Ls) {
  for (int q = 0; q < Ls; ++q) {
    const R m = (R)M[s * Ls + q];
#pragma unroll
    for (int c = 0; c < 2; ++c) out[c] = cfma_r(m, shfl2(v[c], g * Ls + q), out[c]);
  }
}

// h = up + sg A lo of a 4-spinor (A = -i sigma_1, -i sigma_2, -i sigma_3, 1)
template <int MU, class R>
__device__ __forceinline__ void project_mu(const cx<R>* v, R sg, cx<R>* h) {
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    const cx<R> u0 = v[c], u1 = v[3 + c], l0 = v[6 + c], l1 = v[9 + c];
    if constexpr (MU == 0) {
      h[c] = cfma_r(-sg, mul_i(l1), u0);
      h[3 + c] = cfma_r(-sg, mul_i(l0), u1);
    } else if constexpr (MU == 1) {
      h[c] = cfma_r(-sg, l1, u0);
      h[3 + c] = cfma_r(sg, l0, u1);
    } else if constexpr (MU == 2) {
      h[c] = cfma_r(-sg, mul_i(l0), u0);
      h[3 + c] = cfma_r(sg, mul_i(l1), u1);
    } else {
      h[c] = cfma_r(sg, l0, u0);
      h[3 + c] = cfma_r(sg, l1, u1);
    }
  }
}

// FP16S: the arithmetic of the general kernel (packed halves up to the SU(3)
// product, which sums in FP32), one direction per wave.
template <int MU>
__device__ __forceinline__ void project_h(const h2_t* x, bool neg, h2_t* h) {
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    const h2_t u0 = x[c], u1 = x[3 + c], l0 = x[6 + c], l1 = x[9 + c];
    const h2_t il0 = {-l0.y, l0.x}, il1 = {-l1.y, l1.x};
    if constexpr (MU == 0) {
      h[c] = neg ? u0 + il1 : u0 - il1;
      h[3 + c] = neg ? u1 + il0 : u1 - il0;
    } else if constexpr (MU == 1) {
      h[c] = neg ? u0 + l1 : u0 - l1;
      h[3 + c] = neg ? u1 - l0 : u1 + l0;
    } else if constexpr (MU == 2) {
      h[c] = neg ? u0 + il0 : u0 - il0;
      h[3 + c] = neg ? u1 - il1 : u1 + il1;
    } else {
      h[c] = neg ? u0 - l0 : u0 + l0;
      h[3 + c] = neg ? u1 - l1 : u1 + l1;
    }
  }
}

// the words (Re u, -Im u) and (Im u, Re u) of a half link element
__device__ __forceinline__ unsigned re_word(unsigned w) { return w ^ 0x80000000u; }
__device__ __forceinline__ unsigned im_word(unsigned w) { return (w >> 16) | (w << 16); }

// gv = U h for both half spinors; U: the lane's 9 link words. Ls a multiple of 4
// (mf): the four lanes of a block share the link, on the matrix cores with the
// operands of the general kernel's product; else dot products.
__device__ __forceinline__ void su3_half(const unsigned* U, bool mf, int lane, const h2_t* h, cx<float>* gv) {
  if (mf) {
    const bool second = (lane & 2) != 0, im = (lane & 1) != 0;
    unsigned t[3], b[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      const unsigned ut = second ? U[3 + k] : U[k], ub = U[6 + k];
      t[k] = im ? im_word(ut) : re_word(ut);
      b[k] = im ? im_word(ub) : re_word(ub);
    }
    su3_mfma_rows(h4_of(t[0], t[1]), h4_of(t[2], t[1]), h4_of(b[0], b[1]), h4_of(b[2], b[1]), h, gv);
    return;
  }
#pragma unroll
  for (int k = 0; k < 2; ++k)
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      float re = 0.f, im = 0.f;
#pragma unroll
      for (int j = 0; j < 3; ++j) {
        const unsigned u = U[c * 3 + j];
        re = __builtin_amdgcn_fdot2(__builtin_bit_cast(h2_t, re_word(u)), h[k * 3 + j], re, false);
        im = __builtin_amdgcn_fdot2(__builtin_bit_cast(h2_t, im_word(u)), h[k * 3 + j], im, false);
      }
      gv[k * 3 + c] = {re, im};
    }
}

// the two half words and the site scale of pair q
struct Pair16 {
  uint2 w;
  float sc;
};
__device__ __forceinline__ size_t pair16_idx(const FD& f, int r, int q, int s, int i) {
  return 2 * qidx16(f, r, q >> 1, s, i) + (q & 1);  // in units of 8 bytes
}
__device__ __forceinline__ Pair16 ld_pair16(const void* base, const FD& f, int r, int q, int s, int i) {
  return {((const uint2*)base)[pair16_idx(f, r, q, s, i)], scale_ptr(base, f)[sidx(f, r, s, i)]};
}
__device__ __forceinline__ cx<float> half_cx(unsigned w) {
  const h2_t h = __builtin_bit_cast(h2_t, w);
  return {(float)h.x, (float)h.y};
}

template <int P, int ROLE>
__global__ void __launch_bounds__(64 * SMW) hop_small_kernel(HopArgs a) {
  using RT = RoleT<ROLE>;
  using R = typename ST<P>::R;
  static_assert(P != P16 || RT::OM != O_ADDZ, "sources and true residuals are FP64");
  constexpr bool FIN = ROLE == ROLE_K3 || ROLE == ROLE_D3 || ROLE == ROLE_K1T || ROLE == ROLE_D1;
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  cx<R>* s_g = (cx<R>*)smem;  // [direction][component of the half spinor][lane]
  __shared__ double s_red[SMW];
  __shared__ float s_max[P == P16 ? 6 * 64 : 1];
  __shared__ float s_unit[P == P16 ? SMW * 64 : 1];  // FP16S: [direction][lane], the half spinors' unit
  __shared__ int s_halt;

  const int Ls = a.Ls, Vh = a.Vh, G = 64 / Ls;
  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  const int g = lane / Ls, s = lane - g * Ls, r = blockIdx.y;
  // a contiguous run of tiles per XCD (work-groups are dealt round-robin)
  const int nblk = (Vh + G - 1) / G, xcd = blockIdx.x % 8;
  // a CG step on the previous launch's partial sums (K3: alpha, K1: beta) runs in
  // a work-group of its own beside the tiles; the others may see a halt flag
  // before or after it is set, and either is right (a right-hand side halted by
  // this step is not used by the next launch)
  if ((int)blockIdx.x == nblk) {
    if constexpr (FIN) fin_block(a.fin_mode, a.fin_partial + (size_t)r * a.fin_nblk, a.fin_nblk, a.fin_S, r, s_red);
    return;
  }
  const int tile = xcd * (nblk / 8) + min(xcd, nblk % 8) + blockIdx.x / 8;
  const int kk = tile * G + g;
  const bool live = g < G && kk < Vh;
  const FD fd = {Ls, Vh, a.nrhs};
  // one read of the halt flag per work-group: every wave takes the same branch
  if (a.halt != nullptr && tid == 0)
    s_halt = __hip_atomic_load(a.halt + r, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  const int site = min(kk, Vh - 1);  // checkerboard order: a table lookup less in front of the gather
  const int n = a.nbr[(size_t)site * 8 + wave];
  // the link and the neighbour, and this wave's pair of the same-site fields,
  // needed after the sum
  const int q = wave;
  const size_t e = eidx(fd, r, q < 6 ? q : 0, s, site);
  cx<R> U[P == P16 ? 1 : 9], v[P == P16 ? 1 : 12], y[2], z[2];
  unsigned Uh[P == P16 ? 9 : 1], vh[P == P16 ? 12 : 1];
  float vsc = 0.f, zsc = 1.f;
  if constexpr (P == P16) {
#pragma unroll
    for (int j = 0; j < 9; ++j) Uh[j] = ((const unsigned*)a.links)[((size_t)site * 8 + wave) * 9 + j];
    vsc = scale_ptr(a.in, fd)[sidx(fd, r, s, n)];
    ld_words16(a.in, fd, r, s, n, vh);
    if (RT::BM != B_NONE && q < 6) {
      const Pair16 t = ld_pair16(a.y, fd, r, q, s, site);
      y[0] = t.sc * half_cx(t.w.x);
      y[1] = t.sc * half_cx(t.w.y);
    }
    if (RT::OM == O_RUPD && q < 6) {
      const Pair16 t = ld_pair16(a.r, fd, r, q, s, site);
      z[0] = half_cx(t.w.x);
      z[1] = half_cx(t.w.y);
      zsc = t.sc;
    }
  } else {
#pragma unroll
    for (int j = 0; j < 9; ++j) U[j] = ld_link<P>(a.links, ((size_t)site * 8 + wave) * 9 + j);
    ld_spinor<P>(a.in, fd, r, s, n, v);
    if (RT::BM != B_NONE && q < 6) ld_pair<P>(a.y, e, y[0], y[1]);
    if (RT::OM == O_ADDZ && q < 6) ld_pair<P>(a.z, e, z[0], z[1]);
    if (RT::OM == O_RUPD && q < 6) ld_pair<P>(a.r, e, z[0], z[1]);
  }
  const R m = (R)a.mop[r], cpd = (R)a.cpd, cmd = (R)a.cmd, qd = cmd * recip(cpd);
  const double* sc = a.scoef + (size_t)r * (SCOEF_HEAD + 2 * Ls);
  const R sk0 = (R)sc[1], us = (R)sc[SCOEF_HEAD + s], a_s = (R)sc[SCOEF_HEAD + Ls + s];
  const int chi = (int)sc[2];
  SCol<R> col;
  col.dn = g * Ls + (s > 0 ? s - 1 : Ls - 1);
  col.up = g * Ls + (s < Ls - 1 ? s + 1 : 0);
  col.fdn = s > 0 ? R(1) : -m;
  col.fup = s < Ls - 1 ? R(1) : -m;
  col.plus = q < 3;
  if (a.halt != nullptr) {
    __syncthreads();
    if (s_halt != 0) return;
  }

  // direction `wave`: (D~ in)/(c+d) of the neighbour, projected, times the link;
  // the premix factor rounds once, from FP64 (cmd * recip(cpd) in R is up to 2 ulp off)
  const R sg = ((wave < 4) != RT::DAG) ? R(-1) : R(1);
  const R qx = (R)(a.cmd / a.cpd);
  if constexpr (P == P16) {
    // the premix in units of the largest of the three site scales involved
    h2_t x[12], h[6];
    float unit = vsc;
    if constexpr (RT::PRE) {
      const float su = __shfl(vsc, col.dn, 64) * (col.fdn * qx), sl = __shfl(vsc, col.up, 64) * (col.fup * qx);
      unit = fmaxf(vsc, fmaxf(fabsf(su), fabsf(sl)));
      unit = unit > 0.f ? unit : 1.f;
      const float inv = recip(unit);
      const _Float16 f0 = (_Float16)(vsc * inv), fu = (_Float16)(su * inv), fl = (_Float16)(sl * inv);
#pragma unroll
      for (int c = 0; c < 12; ++c) {
        const unsigned t = __shfl(vh[c], c < 6 ? col.dn : col.up, 64);
        x[c] = (c < 6 ? fu : fl) * __builtin_bit_cast(h2_t, t) + f0 * __builtin_bit_cast(h2_t, vh[c]);
      }
    } else {
#pragma unroll
      for (int c = 0; c < 12; ++c) x[c] = __builtin_bit_cast(h2_t, vh[c]);
    }
    const bool neg = sg < R(0);
    switch (wave & 3) {
      case 0: project_h<0>(x, neg, h); break;
      case 1: project_h<1>(x, neg, h); break;
      case 2: project_h<2>(x, neg, h); break;
      default: project_h<3>(x, neg, h); break;
    }
    cx<float> gv[6];
    su3_half(Uh, Ls % 4 == 0, lane, h, gv);
#pragma unroll
    for (int c = 0; c < 6; ++c) s_g[(wave * 6 + c) * 64 + lane] = gv[c];
    s_unit[wave * 64 + lane] = unit;
  } else {
    if constexpr (RT::PRE) {
#pragma unroll
      for (int c = 0; c < 12; ++c) {
        const cx<R> t = shfl2(v[c], c < 6 ? col.dn : col.up);
        v[c] = cfma_r((c < 6 ? col.fdn : col.fup) * qx, t, v[c]);
      }
    }
    cx<R> h[6];
    switch (wave & 3) {
      case 0: project_mu<0>(v, sg, h); break;
      case 1: project_mu<1>(v, sg, h); break;
      case 2: project_mu<2>(v, sg, h); break;
      default: project_mu<3>(v, sg, h); break;
    }
#pragma unroll
    for (int k = 0; k < 2; ++k)
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        cx<R> t = cmul(U[c * 3], h[k * 3]);
        t = cfma(U[c * 3 + 1], h[k * 3 + 1], t);
        t = cfma(U[c * 3 + 2], h[k * 3 + 2], t);
        s_g[(wave * 6 + k * 3 + c) * 64 + lane] = t;
      }
  }
  __syncthreads();

  double nrm = 0.0;
  cx<R> w[2];
  if (q < 6) {
    // the leading factor: -1/2, the (c+d) of D~ on the input, and the
    // epilogue's sign, (c+d) and normalisation
    R fold = RT::PRE ? R(-0.5) * cpd : R(-0.5);
    if constexpr (RT::AM == A_NEG) fold *= R(-1);
    if constexpr (RT::AM == A_DTT || RT::AM == A_MATDT || RT::AM == A_DMINV || RT::AM == A_MINVDT) fold *= cpd;
    if constexpr (RT::AM == A_NDTT) fold *= -cpd;
    constexpr bool SINV = RT::AM == A_DMINV || RT::AM == A_MINVDT;
    if constexpr (SINV) fold *= minv_norm<R>((R)a.bee, (R)a.cee, m, Ls);
    R vscale = R(1);
    if constexpr (RT::OM == O_RUPD) vscale = -(R)a.alpha[r];
    fold *= vscale;

    // the pair's components of sum over directions [g ; sg A^dag g]; in FP16S each
    // direction's unit times the leading factor scales its half spinor as it is added
    R k[P == P16 ? 8 : 1];
    if constexpr (P == P16)
#pragma unroll
      for (int d = 0; d < 8; ++d) k[d] = s_unit[d * 64 + lane] * fold;
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      const int c = 2 * q + t, spin = c / 3, cc = c - 3 * spin;
      cx<R> acc = {R(0), R(0)};
      if (spin < 2) {
#pragma unroll
        for (int d = 0; d < 8; ++d) {
          const cx<R> u = s_g[(d * 6 + spin * 3 + cc) * 64 + lane];
          acc = P == P16 ? cfma_r(k[P == P16 ? d : 0], u, acc) : acc + u;
        }
      } else {
        const bool hi = spin == 3;
#pragma unroll
        for (int d = 0; d < 8; ++d) {
          const int mu = d & 3;
          // A^dag g: mu 0 (i g1, i g0), 1 (g1, -g0), 2 (i g0, -i g1), 3 (g0, g1)
          const bool neg = ((d < 4) != RT::DAG) != ((mu == 1 || mu == 2) && hi);
          const int half = (mu < 2) != hi ? 1 : 0;
          cx<R> u = s_g[(d * 6 + half * 3 + cc) * 64 + lane];
          if (mu == 0 || mu == 2) u = mul_i(u);
          const R f = P == P16 ? k[P == P16 ? d : 0] : R(1);
          acc = cfma_r(neg ? -f : f, u, acc);
        }
      }
      w[t] = P == P16 ? acc : fold * acc;
    }

    const bool shifted = sk0 != R(0) && (chi > 0) == col.plus;  // the shift acts on this chirality
    const int star = col.plus ? Ls - 1 : 0, star_lane = g * Ls + star;
    if constexpr (RT::AM == A_DTT || RT::AM == A_NDTT || RT::AM == A_MATDT || RT::AM == A_MINVDT)
      lacc2<R, true>(w, w, col, qd);
    if constexpr (SINV) {
      const R rho = (R)a.cee * recip((R)a.bee);
      if constexpr (RT::AM == A_MINVDT) {
        if (shifted) {  // z_{s*} += sum_s a_s z_s
#pragma unroll
          for (int t = 0; t < 2; ++t) {
            const cx<R> sum = col_sum<R>(a_s * w[t], g, Ls);
            if (s == star) w[t] = w[t] + sum;
          }
        }
        series2<R, true>(w, s, g, Ls, rho, m, col.plus);
      } else {
        series2<R, false>(w, s, g, Ls, rho, m, col.plus);
        if (shifted) {  // z += a z_{s*}
#pragma unroll
          for (int t = 0; t < 2; ++t) w[t] = cfma_r(a_s, shfl2(w[t], star_lane), w[t]);
        }
      }
    }
    const size_t msz = (size_t)Ls * Ls;
    const double* mats = a.mats + ((size_t)r * NMAT * 2 + (col.plus ? 0 : 1)) * msz;
    if constexpr (RT::AM == A_MAT || RT::AM == A_MATDT) {
      const cx<R> src[2] = {w[0], w[1]};
      w[0] = w[1] = {R(0), R(0)};
      dense2<R>(mats + (size_t)a.matA * 2 * msz, src, w, s, g, Ls);
    }
    if constexpr (RT::AM == A_DMINV) lacc2<R, false>(w, w, col, qd);
    if constexpr (RT::BM == B_DENSE) {
#pragma unroll
      for (int t = 0; t < 2; ++t) y[t] = vscale * y[t];
      dense2<R>(mats + (size_t)a.matB * 2 * msz, y, w, s, g, Ls);
    } else if constexpr (RT::BM != B_NONE) {
      R yn = vscale;
      if constexpr (RT::BM == B_MEE_DTI) {
        series2<R, false>(y, s, g, Ls, -qd, m, col.plus);
        yn *= dtinv_norm<R>(cpd, cmd, m, Ls);
      }
      const R bee = (R)a.bee * yn, cee = (R)a.cee * yn;
#pragma unroll
      for (int t = 0; t < 2; ++t) w[t] = cfma_r(bee, y[t], w[t]);
      lacc2<R, RT::BM == B_MEET>(w, y, col, -cee);
      if (shifted) {
        const R sk = sk0 * yn;
#pragma unroll
        for (int t = 0; t < 2; ++t) {
          if constexpr (RT::BM == B_MEET) {  // sk e_{s*} u^T y
            const cx<R> sum = col_sum<R>(us * y[t], g, Ls);
            if (s == star) w[t] = cfma_r(sk, sum, w[t]);
          } else {  // sk u e_{s*}^T y
            w[t] = cfma_r(sk * us, shfl2(y[t], star_lane), w[t]);
          }
        }
      }
    }
    if constexpr (RT::OM == O_ADDZ) {
#pragma unroll
      for (int t = 0; t < 2; ++t) w[t] = z[t] - w[t];
    } else if constexpr (RT::OM == O_RUPD) {  // w carries -alpha
#pragma unroll
      for (int t = 0; t < 2; ++t) w[t] = P == P16 ? cfma_r((R)zsc, z[t], w[t]) : z[t] + w[t];
    }
    if constexpr (P == P16) {
      s_max[q * 64 + lane] = fmaxf(fmaxf(fabsf(w[0].r), fabsf(w[0].i)), fmaxf(fabsf(w[1].r), fabsf(w[1].i)));
    } else if (live) {
      st_pair<P>(RT::OM == O_RUPD || RT::OM == O_STORE_R ? a.r : a.out, e, w[0], w[1]);
      if constexpr (RT::NRM)
#pragma unroll
        for (int t = 0; t < 2; ++t) nrm += (double)w[t].r * w[t].r + (double)w[t].i * w[t].i;
    }
  }
  if constexpr (P == P16) {  // the encoding, and |v|^2 from it, as st_spinor16
    __syncthreads();
    if (q < 6 && live) {
      float mx = 0.f;
#pragma unroll
      for (int k = 0; k < 6; ++k) mx = fmaxf(mx, s_max[k * 64 + lane]);
      const float inv = mx > 0.f ? recip(mx) : 0.f;
      unsigned hw[2];
      float ns = 0.f;
#pragma unroll
      for (int t = 0; t < 2; ++t) {
        const float xr = (float)w[t].r * inv, xi = (float)w[t].i * inv;
        ns = fma(xi, xi, fma(xr, xr, ns));
        const h2_t h = {(_Float16)xr, (_Float16)xi};
        hw[t] = __builtin_bit_cast(unsigned, h);
      }
      void* dst = RT::OM == O_RUPD || RT::OM == O_STORE_R ? a.r : a.out;
      ((uint2*)dst)[pair16_idx(fd, r, q, s, site)] = make_uint2(hw[0], hw[1]);
      if (q == 0) ((float*)scale_ptr(dst, fd))[sidx(fd, r, s, site)] = mx;
      if constexpr (RT::NRM) nrm = (double)mx * (double)mx * (double)ns;
    }
  }
  if constexpr (RT::NRM) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) nrm += __shfl_xor(nrm, off, 64);
    if (lane == 0) s_red[wave] = nrm;
    __syncthreads();
    if (tid == 0) {
      double t = 0.0;
      for (int k = 0; k < 6; ++k) t += s_red[k];
      a.partial[(size_t)r * nblk + blockIdx.x] = t;
    }
  }
}

template <int P, int ROLE>
int launch_small_t(const HopArgs& a, hipStream_t st) {
  const int G = 64 / a.Ls;
  const size_t lds = sizeof(cx<typename ST<P>::R>) * SMW * 6 * 64;  // 48 KiB in FP64
  hipLaunchKernelGGL((hop_small_kernel<P, ROLE>), dim3((a.Vh + G - 1) / G + (a.fin_partial ? 1 : 0), a.nrhs),
                     dim3(64 * SMW), lds, st, a);
  return hipGetLastError() == hipSuccess ? EOFA_OK : EOFA_ERR_HIP;
}

// the roles that the library launches in each precision
template <int P>
int launch_small_p(int role, const HopArgs& a, hipStream_t st) {
#define EOFA_CASE(X) \
  case X: return launch_small_t<P, X>(a, st);
  switch (role) {
    EOFA_CASE(ROLE_DSLASH)
    EOFA_CASE(ROLE_DSLASH_DAG)
    EOFA_CASE(ROLE_K1T)
    EOFA_CASE(ROLE_K2T)
    EOFA_CASE(ROLE_K3)
    EOFA_CASE(ROLE_K4)
    EOFA_CASE(ROLE_K4S)
    EOFA_CASE(ROLE_D1)
    EOFA_CASE(ROLE_D2)
    EOFA_CASE(ROLE_D3)
    EOFA_CASE(ROLE_D4)
    EOFA_CASE(ROLE_D4S)
  }
  if constexpr (P != P16) switch (role) {  // the operator on a plain field
      EOFA_CASE(ROLE_K1)
      EOFA_CASE(ROLE_K2)
    }
  if constexpr (P == P64) switch (role) {  // sources and true residuals
      EOFA_CASE(ROLE_SRC)
      EOFA_CASE(ROLE_RES)
      EOFA_CASE(ROLE_FULLRES)
      EOFA_CASE(ROLE_DSRC)
      EOFA_CASE(ROLE_DRES)
      EOFA_CASE(ROLE_DFULLRES)
    }
#undef EOFA_CASE
  return EOFA_ERR_INVALID;
}

}  // namespace

int launch_hop_small(int prec, int role, const HopArgs& a, hipStream_t st) {
  switch (prec) {
    case P64: return launch_small_p<P64>(role, a, st);
    case P32: return launch_small_p<P32>(role, a, st);
  }
  return launch_small_p<P16>(role, a, st);
}

}  // namespace eofa
