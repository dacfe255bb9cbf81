// What the two forms of the hop kernel share (kernels.hip, hop_small.hip): the
// roles, the normalisations of the structured inverses, the fused CG step.
#pragma once

#include <hip/hip_runtime.h>

#include "device_common.h"
#include "internal.h"

namespace eofa {

// epilogue applied to the hop result h = Dhop (D~ in) of each 5D site:
//   A_ID    v = h              A_NEG  v = -h
//   A_MAT   v = M h            (dense Ls x Ls per chirality, through LDS)
//   A_DTT   v = D~^T h         A_NDTT v = -D~^T h   (structured: lane exchange)
//   A_MATDT v = M D~^T h
//   A_DMINV v = D~ M_ee^-1 h   A_MINVDT v = M_ee^-T D~^T h   (the inverse
//           structured along the column: minv_rows for Ls = 16, minv_cols
//           otherwise; D~ and D~^T by lane exchange)
// plus the same-site term B y:
//   B_MEE   + M_ee y           B_MEET + M_ee^T y    (structured: lane exchange)
//   B_MEE_DTI + M_ee D~^-1 y   (y = p~ = D~ p; D~^-1 a geometric series along s)
enum { A_ID = 0, A_NEG = 1, A_MAT = 2, A_DTT = 3, A_NDTT = 4, A_MATDT = 5, A_DMINV = 6, A_MINVDT = 7 };
enum { B_NONE = 0, B_MEE = 1, B_MEET = 2, B_DENSE = 3, B_MEE_DTI = 4 };
enum { O_STORE = 0, O_ADDZ = 1, O_RUPD = 2, O_STORE_R = 3 };

template <int ROLE>
struct RoleT;
#define EOFA_ROLE(NAME, dag, pre, am, bm, om, nrm)   \
  template <>                                        \
  struct RoleT<NAME> {                               \
    static constexpr bool DAG = dag, PRE = pre;      \
    static constexpr int AM = am;                    \
    static constexpr int BM = bm;                    \
    static constexpr int OM = om;                    \
    static constexpr bool NRM = nrm;                 \
  };
EOFA_ROLE(ROLE_DSLASH, false, true, A_ID, B_NONE, O_STORE, false)
EOFA_ROLE(ROLE_DSLASH_DAG, true, false, A_DTT, B_NONE, O_STORE, false)
EOFA_ROLE(ROLE_K1, false, true, A_DMINV, B_NONE, O_STORE, false)
EOFA_ROLE(ROLE_K2, false, false, A_NEG, B_MEE, O_STORE, true)
EOFA_ROLE(ROLE_K3, true, false, A_MINVDT, B_NONE, O_STORE, false)
EOFA_ROLE(ROLE_K4, true, false, A_NDTT, B_MEET, O_RUPD, true)
EOFA_ROLE(ROLE_K4S, true, false, A_NDTT, B_MEET, O_STORE_R, true)
EOFA_ROLE(ROLE_SRC, false, true, A_ID, B_NONE, O_ADDZ, false)
EOFA_ROLE(ROLE_RES, false, false, A_NEG, B_MEE, O_ADDZ, true)
EOFA_ROLE(ROLE_FULLRES, false, true, A_ID, B_MEE, O_ADDZ, true)
// dense (non-Cayley) form: off-parity blocks Dhop alone, same-parity blocks dense
EOFA_ROLE(ROLE_D1, false, false, A_MAT, B_NONE, O_STORE, false)
EOFA_ROLE(ROLE_D2, false, false, A_NEG, B_DENSE, O_STORE, true)
EOFA_ROLE(ROLE_D3, true, false, A_MAT, B_NONE, O_STORE, false)
EOFA_ROLE(ROLE_D4, true, false, A_NEG, B_DENSE, O_RUPD, true)
EOFA_ROLE(ROLE_D4S, true, false, A_NEG, B_DENSE, O_STORE_R, true)
EOFA_ROLE(ROLE_DSRC, false, false, A_ID, B_NONE, O_ADDZ, false)
EOFA_ROLE(ROLE_DRES, false, false, A_NEG, B_DENSE, O_ADDZ, true)
EOFA_ROLE(ROLE_DFULLRES, false, false, A_ID, B_DENSE, O_ADDZ, true)
// the search direction held as p~ = D~ p: no premix in K1, D~^-1 on the same-site term of K2
EOFA_ROLE(ROLE_K1T, false, false, A_DMINV, B_NONE, O_STORE, false)
EOFA_ROLE(ROLE_K2T, false, false, A_NEG, B_MEE_DTI, O_STORE, true)
#undef EOFA_ROLE

// 1/x: the hardware reciprocal (1 ulp) in FP32, a division in FP64
template <class R>
__device__ __forceinline__ R recip(R x) {
  if constexpr (sizeof(R) == 4)
    return __builtin_amdgcn_rcpf(x);
  else
    return R(1) / x;
}

// the normalisations the structured inverses leave to their callers:
// 1/(bee (1 + m rho^Ls)), rho = cee/bee, of M_ee^-1 (unshifted part), and
// 1/((c+d)(1 + m q^Ls)), q = (c-d)/(c+d), of D~^-1
template <class R>
__device__ __forceinline__ R power_ls(R x, int Ls) {  // x^Ls by squaring
  R p = R(1), b = x;
  for (int e = Ls; e > 0; e >>= 1) {
    if (e & 1) p *= b;
    b *= b;
  }
  return p;
}
template <class R>
__device__ __forceinline__ R minv_norm(R bee, R cee, R m, int Ls) {
  return recip(bee * (R(1) + m * power_ls(cee * recip(bee), Ls)));
}
template <class R>
__device__ __forceinline__ R dtinv_norm(R cpd, R cmd, R m, int Ls) {
  return recip(cpd * (R(1) + m * power_ls(cmd * recip(cpd), Ls)));
}

typedef _Float16 h4_t __attribute__((ext_vector_type(4)));
typedef float f4_t __attribute__((ext_vector_type(4)));
typedef unsigned u2_t __attribute__((ext_vector_type(2)));
__device__ __forceinline__ h4_t h4_of(unsigned lo, unsigned hi) { return __builtin_bit_cast(h4_t, u2_t{lo, hi}); }
__device__ __forceinline__ h4_t h4_of(h2_t lo, h2_t hi) { return __builtin_shufflevector(lo, hi, 0, 1, 2, 3); }

// the two projected half spinors h[0..2], h[3..5] times the rows of U that this
// lane holds: A00, A01 of colours 0 and 1, A10, A11 of colour 2
__device__ __forceinline__ void su3_mfma_rows(h4_t A00, h4_t A01, h4_t A10, h4_t A11, const h2_t* h, cx<float>* gv) {
  const h2_t z2 = {(_Float16)0.f, (_Float16)0.f};
  const f4_t z4 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int k = 0; k < 2; ++k) {
    const h4_t B0 = h4_of(h[k * 3], h[k * 3 + 1]), B1 = h4_of(h[k * 3 + 2], z2);
    f4_t t = __builtin_amdgcn_mfma_f32_4x4x4f16(A00, B0, z4, 0, 0, 0);
    t = __builtin_amdgcn_mfma_f32_4x4x4f16(A01, B1, t, 0, 0, 0);
    f4_t b = __builtin_amdgcn_mfma_f32_4x4x4f16(A10, B0, z4, 0, 0, 0);
    b = __builtin_amdgcn_mfma_f32_4x4x4f16(A11, B1, b, 0, 0, 0);
    gv[k * 3] = {t[0], t[1]};
    gv[k * 3 + 1] = {t[2], t[3]};
    gv[k * 3 + 2] = {b[0], b[1]};
  }
}

// one CG scalar step for right-hand side r from the reduced sum
static __device__ void finalize_step(int mode, double sum, const CgState& S, int r, double* out) {
  if (mode == FIN_NORM) {
    out[r] = sum;
    return;
  }
  if (mode == FIN_INIT) {
    S.rr[r] = sum;
    S.stop[r] = S.tol2[r] * sum;
    S.guard[r] *= sum;
    S.iter[r] = 0;
    S.u2run[r] = 0;
    S.breakdown[r] = 0;
    S.halt[r] = (sum == 0.0 || S.max_iter[r] <= 0) ? 1 : 0;
    if (!isfinite(sum)) {
      S.breakdown[r] = 1;
      S.halt[r] = 1;
    }
    return;
  }
  if (mode == FIN_ALPHA) {
    if (S.halt[r]) return;
    S.ww[r] = sum;
    if (!(sum > 0.0) || !isfinite(sum)) {
      S.breakdown[r] = 1;
      S.halt[r] = 1;
      S.alpha[r] = 0.0;
      return;
    }
    S.alpha[r] = S.rr[r] / sum;
    return;
  }
  // FIN_BETA
  if (S.halt[r]) {
    S.u2run[r] = 0;
    return;
  }
  const double rrn = sum;
  S.beta[r] = rrn / S.rr[r];
  S.rr[r] = rrn;
  S.iter[r] += 1;
  S.u2run[r] = 1;
  if (!isfinite(rrn)) {
    S.breakdown[r] = 1;
    S.halt[r] = 1;
    S.u2run[r] = 0;
  } else if (rrn <= S.stop[r] || S.iter[r] >= S.max_iter[r]) {
    S.halt[r] = 1;
  } else if (S.guard[r] > 0.0 && rrn > S.guard[r]) {
    S.halt[r] = 1;
    S.breakdown[r] = 2;
  }
}

// A CG step fused into a hop launch, run by one work-group (which one: see HopArgs):
// the previous launch's nblk partial sums of right-hand side r, reduced by the
// whole work-group in a fixed order (8 independent sums per
// thread, then lanes, then waves), then finalize_step on thread 0. red: one
// double per wave.
__device__ __forceinline__ void fin_block(int mode, const double* __restrict__ pr, int nblk, const CgState& S, int r,
                                          double* red) {
  const int tid = threadIdx.x, nthr = blockDim.x;
  double acc[8];
#pragma unroll
  for (int k = 0; k < 8; ++k) acc[k] = 0.0;
  for (int j0 = tid; j0 < nblk; j0 += 8 * nthr) {
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      const int j = j0 + k * nthr;
      if (j < nblk) acc[k] += pr[j];
    }
  }
#pragma unroll
  for (int w = 4; w > 0; w >>= 1)
#pragma unroll
    for (int k = 0; k < w; ++k) acc[k] += acc[k + w];
  double t = acc[0];
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) t += __shfl_xor(t, off, 64);
  if ((tid & 63) == 0) red[tid >> 6] = t;
  __syncthreads();
  if (tid == 0) {
    double sum = 0.0;
    for (int w = 0; w < (nthr + 63) / 64; ++w) sum += red[w];
    finalize_step(mode, sum, S, r, nullptr);
  }
  __syncthreads();
}

}  // namespace eofa
