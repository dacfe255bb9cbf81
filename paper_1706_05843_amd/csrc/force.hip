// Link derivative of the hopping term and the EOFA pseudofermion force
// (Sec. IV C, eqn eofa_force).
//
// For 5D fields a, b and one link (x, mu), the derivative of
// a^dag Dhop b along U_mu(x) -> e^{s T} U_mu(x) at s = 0 is, for every
// traceless anti-Hermitian T (Dhop: overall -1/2, eqn Ddwf),
//   -1/2 sum_s [ a^dag(x,s) (1 - g_mu) T U b(x+mu,s) - a^dag(x+mu,s) (1 + g_mu) U^dag T b(x,s) ]
//   = Tr(T y),   y = -1/2 U B1 + 1/2 B2 U^dag,
//   B1 = sum_s Tr_spin[(1 - g_mu) b(x+mu,s) a(x,s)^dag],
//   B2 = sum_s Tr_spin[(1 + g_mu) b(x,s) a(x+mu,s)^dag]
// (U with the boundary phase of the link). In the chiral basis
// g_mu = [[0, A], [A^dag, 0]], so Tr_spin[(1 + sg g_mu) v w^dag] is the sum over
// the two components of h_v h_w^dag with h = up + sg A lo: only projected
// 2-spinors enter.
//
// Layouts: fields canonical complex128 [Ls][T][Z][Y][X][4][3]; links the
// packed FP64 per-parity tables (forward direction mu of site i of parity p
// at ((i * 8 + mu) * 9), phase included); y and the force canonical
// complex128 [4][T][Z][Y][X][3][3].
#include <hip/hip_runtime.h>

#include "device_common.h"
#include "force_internal.h"

namespace eofa {

namespace {

__device__ __forceinline__ size_t lex_of(const int L[4], const int x[4]) {
  return (((size_t)x[3] * L[2] + x[2]) * L[1] + x[1]) * L[0] + x[0];
}

// Bound by the loads of a and b: each site's spinors serve four links forward
// and four backward. A work-group takes DV_T consecutive sites and all Ls; its
// four waves take one direction each, a lane pair one link, a lane one of the
// two projected components k (which needs spin k and its partner under g_mu
// alone: half a spinor, half the 36 accumulators). Per s the tile's a and b and
// those of the neighbours outside the tile go through LDS once, read by
// neighbouring lanes (16 bytes each of a 192-byte spinor), while the previous s
// is computed. 16^3 x 32 x 16: 315 us (3.0 TB/s of the compulsory bytes; with the
// tiles in plain order 369), 24^3 x 32 x 12 864 us (1028). One thread per site and
// direction, reading its four spinors per s from memory 192 bytes a lane, took
// 1243 and 3408 us.
constexpr int DV_T = 32;                  // sites per work-group
constexpr int DV_SLOTS = 5 * DV_T;        // the tile, then DV_T neighbours per direction
constexpr int DV_ELEMS = DV_SLOTS * 12;   // complex numbers of one field staged per s
constexpr int DV_ITER = (DV_ELEMS + 255) / 256;

__device__ __forceinline__ unsigned block_of(unsigned n) { return n % 4 == 0 ? 4 : (n % 2 == 0 ? 2 : 1); }

__global__ void __launch_bounds__(256) dhop_deriv_kernel(DerivArgs d) {
  extern __shared__ d2v_t s_f[];  // [2][DV_ELEMS]: a, then b
  __shared__ unsigned s_site[DV_SLOTS];
  __shared__ int s_nbr[4 * DV_T];   // slot of the site's neighbour x + mu
  __shared__ int s_n[3];
  const size_t V = (size_t)d.L[0] * d.L[1] * d.L[2] * d.L[3];
  const int tid = threadIdx.x, mu = tid >> 6, lane = tid & 63, j = lane >> 1, k = lane & 1;
  // a contiguous run of tiles per XCD (work-groups are dealt round-robin)
  const int nblk = gridDim.x, xcd = blockIdx.x % 8;
  unsigned tile = xcd * (nblk / 8) + min(xcd, nblk % 8) + blockIdx.x / 8;
  // in blocks of up to 4 tiles of a plane x 4 z x 4 t, about the tiles an XCD has
  // in flight, so that most z and t neighbours are fetched once per XCD
  if (nblk >= 512 && d.L[0] * d.L[1] % DV_T == 0) {
    const unsigned np = d.L[0] * d.L[1] / DV_T, bp = block_of(np), bz = block_of(d.L[2]), bt = block_of(d.L[3]);
    const unsigned in = tile % (bp * bz * bt), blk = tile / (bp * bz * bt);
    const unsigned nbp = np / bp, nbz = d.L[2] / bz;
    const unsigned p = blk % nbp * bp + in % bp, z = blk / nbp % nbz * bz + in / bp % bz;
    const unsigned t = blk / (nbp * nbz) * bt + in / (bp * bz);
    tile = (t * d.L[2] + z) * np + p;
  }
  const unsigned base = tile * DV_T;
  const unsigned nV = (unsigned)V;
  // slots: the tile's sites, then the neighbours outside it, without gaps
  {
    unsigned ln = 0;
    bool outside = false;
    if (tid < 4 * DV_T) {
      const int m = tid / DV_T, q = tid - m * DV_T;
      const unsigned lx = min(base + q, nV - 1);
      int x[4];
      unsigned rest = lx;
      for (int t = 0; t < 4; ++t) {
        x[t] = rest % d.L[t];
        rest /= d.L[t];
      }
      x[m] = x[m] + 1 == d.L[m] ? 0 : x[m] + 1;
      ln = (unsigned)lex_of(d.L, x);
      outside = ln < base || ln >= min(base + DV_T, nV);
      if (m == 0) s_site[q] = lx;
    }
    const unsigned long long mask = __ballot(outside);
    if (lane == 0 && mu < 2) s_n[mu] = __popcll(mask);
    __syncthreads();
    if (tid < 4 * DV_T) {
      const int slot = DV_T + (mu ? s_n[0] : 0) + __popcll(mask & ((1ull << lane) - 1));
      s_nbr[tid] = outside ? slot : (int)(ln - base);
      if (outside) s_site[slot] = ln;
    }
    __syncthreads();
  }
  const int nelem = (DV_T + s_n[0] + s_n[1]) * 12;
  // this thread's staged elements: offset within a field's s slice
  unsigned off[DV_ITER];
#pragma unroll
  for (int t = 0; t < DV_ITER; ++t) {
    const int e = min(t * 256 + tid, nelem - 1), slot = e / 12, c = e - slot * 12;
    off[t] = s_site[slot] * 12u + c;
  }
  d2v_t ra[DV_ITER], rb[DV_ITER];
#pragma unroll
  for (int t = 0; t < DV_ITER; ++t) ra[t] = rb[t] = d2v_t{0.0, 0.0};
  auto fetch = [&](int s) {
    const d2v_t* pa = (const d2v_t*)d.a + (size_t)(d.g5r5_a ? d.Ls - 1 - s : s) * V * 12;
    const d2v_t* pb = (const d2v_t*)d.b + (size_t)s * V * 12;
#pragma unroll
    for (int t = 0; t < DV_ITER; ++t)
      if (t * 256 < nelem) {  // uniform
        ra[t] = pa[off[t]];
        rb[t] = pb[off[t]];
      }
  };
  const unsigned lx = base + j;
  const bool live = lx < nV;
  const int slot0 = j * 12, slot1 = s_nbr[mu * DV_T + j] * 12;
  // A lo of component k: partner spin, whether times i, and its sign
  // (A = -i sigma_1, -i sigma_2, -i sigma_3, 1)
  const int part = (mu < 2 ? 3 - k : 2 + k) * 3, own = k * 3;
  const bool times_i = mu == 0 || mu == 2;
  const double sgn = mu == 0 ? -1.0 : mu == 3 ? 1.0 : k ? 1.0 : -1.0;
  const double sgn_a = d.g5r5_a ? -sgn : sgn;  // gamma_5 on a's lower spins
  cx<double> B1[9], B2[9];
#pragma unroll
  for (int q = 0; q < 9; ++q) B1[q] = B2[q] = {0.0, 0.0};
  fetch(0);
  for (int s = 0; s < d.Ls; ++s) {
    __syncthreads();
#pragma unroll
    for (int t = 0; t < DV_ITER; ++t) {
      const int e = t * 256 + tid;
      if (e < nelem) {
        s_f[e] = ra[t];
        s_f[DV_ELEMS + e] = rb[t];
      }
    }
    __syncthreads();
    if (s + 1 < d.Ls) fetch(s + 1);
    if (!live) continue;
    // up + sg A lo of component k, three colours
    auto project = [&](const d2v_t* v, double sg, cx<double>* h) {
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        const d2v_t u = v[own + c], l = v[part + c];
        const double zr = times_i ? -l.y : l.x, zi = times_i ? l.x : l.y;
        h[c] = {fma(sg, zr, u.x), fma(sg, zi, u.y)};
      }
    };
    auto outer = [](const cx<double>* v, const cx<double>* w, cx<double>* B) {
#pragma unroll
      for (int r = 0; r < 3; ++r)
#pragma unroll
        for (int c = 0; c < 3; ++c) {  // v conj(w)
          cx<double>& t = B[r * 3 + c];
          t.r = fma(v[r].r, w[c].r, fma(v[r].i, w[c].i, t.r));
          t.i = fma(v[r].i, w[c].r, fma(-v[r].r, w[c].i, t.i));
        }
    };
    cx<double> v[3], w[3];
    project(s_f + DV_ELEMS + slot1, -sgn, v);  // B1: (1 - g_mu) b(x+mu) a(x)^dag
    project(s_f + slot0, -sgn_a, w);
    outer(v, w, B1);
    project(s_f + DV_ELEMS + slot0, sgn, v);  // B2: (1 + g_mu) b(x) a(x+mu)^dag
    project(s_f + slot1, sgn_a, w);
    outer(v, w, B2);
  }
  // the two components' sums (every lane takes part in the exchange)
#pragma unroll
  for (int q = 0; q < 9; ++q) {
    B1[q].r += __shfl_xor(B1[q].r, 1, 64);
    B1[q].i += __shfl_xor(B1[q].i, 1, 64);
    B2[q].r += __shfl_xor(B2[q].r, 1, 64);
    B2[q].i += __shfl_xor(B2[q].i, 1, 64);
  }
  if (!live) return;
  int x[4];
  unsigned rest = lx;
  for (int t = 0; t < 4; ++t) {
    x[t] = rest % d.L[t];
    rest /= d.L[t];
  }
  const int p = (x[0] + x[1] + x[2] + x[3]) & 1;
  const double2* Up = d.links[p] + ((size_t)(lx / 2) * 8 + mu) * 9;
  cx<double> U[9];
#pragma unroll
  for (int q = 0; q < 9; ++q) U[q] = {Up[q].x, Up[q].y};
  // y = coef (-1/2 U B1 + 1/2 B2 U^dag); lane k stores every second entry
  double2* out = d.y + ((size_t)mu * V + lx) * 9;
#pragma unroll
  for (int r = 0; r < 3; ++r)
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      cx<double> t1 = {0.0, 0.0}, t2 = {0.0, 0.0};
#pragma unroll
      for (int q = 0; q < 3; ++q) {
        t1 = cfma(U[r * 3 + q], B1[q * 3 + c], t1);
        const cx<double> ud = {U[c * 3 + q].r, -U[c * 3 + q].i};  // (U^dag)[q][c]
        t2 = cfma(B2[r * 3 + q], ud, t2);
      }
      if (((r * 3 + c) & 1) != k) continue;
      const cx<double> yv = {d.coef * 0.5 * (t2.r - t1.r), d.coef * 0.5 * (t2.i - t1.i)};
      double2 o = d.accumulate ? out[r * 3 + c] : make_double2(0.0, 0.0);
      o.x += yv.r;
      o.y += yv.i;
      out[r * 3 + c] = o;
    }
}

// F = sum_a T^a Re Tr(T^a Y) = -1/4 [(Y - Y^dag) - 1/3 Tr(Y - Y^dag)] for the
// basis T^a = i lambda^a / 2 (Tr T^a T^b = -1/2 delta^ab), in place
__global__ void force_project_kernel(size_t nlinks, double2* y) {
  const size_t k = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= nlinks) return;
  double2* m = y + k * 9;
  cx<double> Z[9];
#pragma unroll
  for (int r = 0; r < 3; ++r)
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      const double2 a = m[r * 3 + c], b = m[c * 3 + r];
      Z[r * 3 + c] = {a.x - b.x, a.y + b.y};  // Y - Y^dag
    }
  const double tr_i = (Z[0].i + Z[4].i + Z[8].i) / 3.0;  // the trace of Y - Y^dag is imaginary
#pragma unroll
  for (int r = 0; r < 3; ++r)
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      cx<double> z = Z[r * 3 + c];
      if (r == c) z.i -= tr_i;
      m[r * 3 + c] = make_double2(-0.25 * z.r, -0.25 * z.i);
    }
}

// G-parity in x on the x-doubled lattice: U2(x') = U(x') for x' < Lx,
// conj(U(x' - Lx)) for Lx <= x' < 2 Lx (the flavour-1 copy)
__global__ void double_gauge_kernel(int Lx, size_t rows, const double2* U, double2* U2) {
  const size_t k = (size_t)blockIdx.x * blockDim.x + threadIdx.x;  // over 4 * rows * 2Lx sites
  const size_t nsite = (size_t)4 * rows * 2 * Lx;
  if (k >= nsite) return;
  const int xd = (int)(k % (2 * Lx));
  const size_t row = k / (2 * Lx);  // (mu, t, z, y)
  const bool flv = xd >= Lx;
  const double2* src = U + (row * Lx + (flv ? xd - Lx : xd)) * 9;
  double2* dst = U2 + k * 9;
#pragma unroll
  for (int c = 0; c < 9; ++c) {
    const double2 v = src[c];
    dst[c] = make_double2(v.x, flv ? -v.y : v.y);
  }
}

// physical force F(x) = F2(x) + conj(F2(x + Lx)) from the doubled-lattice one
__global__ void fold_force_kernel(int Lx, size_t rows, const double2* F2, double2* F) {
  const size_t k = (size_t)blockIdx.x * blockDim.x + threadIdx.x;  // over 4 * rows * Lx links
  if (k >= (size_t)4 * rows * Lx) return;
  const int x = (int)(k % Lx);
  const size_t row = k / Lx;
  const double2* a = F2 + (row * 2 * Lx + x) * 9;
  const double2* b = F2 + (row * 2 * Lx + x + Lx) * 9;
#pragma unroll
  for (int c = 0; c < 9; ++c) F[k * 9 + c] = make_double2(a[c].x + b[c].x, a[c].y - b[c].y);
}

}  // namespace

void launch_double_gauge(int Lx, size_t rows, const void* U, void* U2, hipStream_t st) {
  const size_t n = (size_t)4 * rows * 2 * Lx;
  hipLaunchKernelGGL(double_gauge_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, Lx, rows,
                     (const double2*)U, (double2*)U2);
}

void launch_fold_force(int Lx, size_t rows, const void* F2, void* F, hipStream_t st) {
  const size_t n = (size_t)4 * rows * Lx;
  hipLaunchKernelGGL(fold_force_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, Lx, rows,
                     (const double2*)F2, (double2*)F);
}

void launch_dhop_deriv(const DerivArgs& d, hipStream_t st) {
  const int ntile = (2 * d.Vh + DV_T - 1) / DV_T;
  hipLaunchKernelGGL(dhop_deriv_kernel, dim3(ntile), dim3(256), 2 * DV_ELEMS * sizeof(double2), st, d);
}

void launch_force_project(size_t nlinks, void* y, hipStream_t st) {
  hipLaunchKernelGGL(force_project_kernel, dim3((unsigned)((nlinks + 255) / 256)), dim3(256), 0, st, nlinks,
                     (double2*)y);
}

}  // namespace eofa
