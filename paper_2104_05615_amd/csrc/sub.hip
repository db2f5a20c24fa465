// Preconditioner kernels (Sec. 2.4-2.5): moving the outer residual into the
// centre region C of every virtual subdomain and the inner solution back, and
// the inner CG's vector updates with per-subdomain scalars.  The four hops of
// the local operator A_s run through hop_sub (kernels.hip).
//
// All of them are bound by the fields they stream (4.7 to 5.6 TB/s at 32^3x64;
// a copy reaches 5.0), so the updates are grouped by what has to be read: a
// middle inner step reads and writes 9 fields outside the hops (10 with z
// updated beside r), the restriction writes r_s once (not as r_s and p_s), and
// the last step's z goes from registers into the outer field.  Measured, the
// whole preconditioner: 32^3x64 x 12, FP16, k = 3 19.2 -> 18.2 ms; 16^3x32 x
// 12, FP16, k = 6 3081 -> 2999 us; 16^4 x 16, INT8, k = 6 1701 -> 1661 us.
//
// All kernels here map threads like the site kernels: a block owns ns sites
// of C of one subdomain and all their Ls slices, so per-block partial sums are
// grouped by subdomain as [d][bps].  Batched launches put the RHS in
// blockIdx.y: fields at RHS offsets (Field::at), per-subdomain scalars at
// r * nsub, partials at r * nsub * bps; RHS with mask[r] == 0 are skipped.
#include <stdexcept>
#include <string>

#include "kernels.h"
#include "sitekern.h"

namespace mspcg {

#define LAUNCH_CHECK()                                                                \
  do {                                                                                \
    hipError_t e_ = hipGetLastError();                                                \
    if (e_ != hipSuccess) throw std::runtime_error(std::string("kernel launch: ") +   \
                                                   hipGetErrorString(e_));            \
  } while (0)

struct CSite {
  bool inb, valid;
  int sl, s;
  int64_t blk, d, j, in5;   // in5: index in the per-subdomain C field
};

__device__ __forceinline__ CSite c_site(const SubTables& tc, int ns, int Ls) {
  CSite c;
  const int tid = threadIdx.x;
  c.inb = tid < ns * Ls;
  c.sl = c.inb ? tid / Ls : 0;
  c.s = c.inb ? tid - c.sl * Ls : 0;
  c.blk = xcd_block(blockIdx.x, gridDim.x);
  c.d = (int64_t)tc.fbps.div((uint32_t)c.blk);   // blocks < 2^31
  c.j = (c.blk - c.d * tc.bps) * ns + c.sl;
  c.valid = c.inb && c.j < tc.n_out;
  c.in5 = (c.d * tc.n_out + c.j) * Ls + c.s;
  return c;
}

// global single-parity index of centre site j of subdomain d
__device__ __forceinline__ uint32_t c_global(const SubTables& tc, const Lattice& lat, int64_t d, int64_t j) {
  const short4 o = tc.origin[d];
  const short4 lc = tc.coords[j];
  // centre sites lie inside the subdomain: no wrap needed
  const int g[4] = {o.x + lc.x, o.y + lc.y, o.z + lc.z, o.w + lc.w};
  return lat.index(g);
}

template <typename O, typename I>
__global__ void __launch_bounds__(256)
k_sub_restrict(Field<O> r, Field<I> rs, Field<I> t0, const calc_t<I>* E, Lattice lat, SubTables tc,
               int Ls, int ns, double* partial, const int* mask) {
  using T = calc_t<I>;
  const int rhs = blockIdx.y;
  if (mask && mask[rhs] == 0) return;
  r = r.at(rhs);
  rs = rs.at(rhs);
  t0 = t0.at(rhs);
  partial += (int64_t)rhs * gridDim.x;
  extern __shared__ __align__(16) unsigned char lds_raw[];
  double* red = reinterpret_cast<double*>(lds_raw);
  T* mats = reinterpret_cast<T*>(red + 16);
  T* tile = mats + 2 * Ls * Ls;
  const CSite c = c_site(tc, ns, Ls);
  for (int k = threadIdx.x; k < 2 * Ls * Ls; k += blockDim.x) mats[k] = E[k];
  T v[24];
  if (c.valid) {
    const int64_t g = c_global(tc, lat, c.d, c.j);
    load_site(r, g * Ls + c.s, v);
    store_site(rs, c.in5, v);
  } else {
#pragma unroll
    for (int k = 0; k < 24; ++k) v[k] = 0;
  }
  double loc = 0;
#pragma unroll
  for (int k = 0; k < 24; ++k) loc += (double)v[k] * (double)v[k];
  T* my = tile + c.sl * tile_stride(Ls);
  if (c.inb) tile_put(my, c.s, v);
  __syncthreads();
  if (c.inb) mat5_lds(my, mats, c.s, Ls, v, false);
  if (c.valid) store_site(t0, c.in5, v);
  const double tot = block_sum(loc, red);
  if (threadIdx.x == 0) partial[c.blk] = tot;
}

// sum of the bps partials of subdomain d, by every wavefront in the same fixed
// order (lane-strided, then a butterfly)
__device__ __forceinline__ double sub_sum(const double* partial, int bps, int64_t d) {
  double S = 0;
  for (int b = threadIdx.x & 63; b < bps; b += 64) S += partial[d * bps + b];
  for (int off = 32; off > 0; off >>= 1) S += __shfl_xor(S, off);
  return S;
}

// Per-subdomain scalars of the inner CG, evaluated in the kernel that uses
// them: every wavefront sums the bps partials in one fixed order, so each gets
// the same value to the bit without a barrier, and the field loads of the
// kernel need not wait for it.  Thread 0 of the block holding the subdomain's
// first site block also stores the new state.  Other wavefronts may read
// `active` while that thread clears it, but it is cleared only where every
// reader takes the same decision from the same sum; rho is read from one array
// and written to another.  Call from every lane of the wavefront.
//
// alpha = rho / <p, q> (0 where the subdomain has stopped or <p, q> is not
// positive).  With rr0 (the first step) rho is the sum of those partials of
// |r_s|^2, and rho and active are stored too.
__device__ __forceinline__ double fused_alpha(const double* pq, const double* rr0, int bps, int64_t d, bool first_blk,
                                              double* rho, double* alpha, int* active) {
  const double S = sub_sum(pq, bps, d);
  const double r = rr0 ? sub_sum(rr0, bps, d) : rho[d];
  const bool act = rr0 ? r > 0.0 : active[d] != 0;
  const bool ok = act && S > 0.0 && isfinite(S);
  const double v = ok ? r / S : 0.0;
  if (first_blk && threadIdx.x == 0) {
    alpha[d] = v;
    if (rr0) {
      rho[d] = r;
      active[d] = ok ? 1 : 0;
    } else if (!ok) {
      active[d] = 0;
    }
  }
  return v;
}

// beta = |r_s|^2 / rho; rho_next = |r_s|^2
__device__ __forceinline__ double fused_beta(const double* rr, int bps, int64_t d, bool first_blk, const double* rho,
                                             double* rho_next, double* beta, int* active) {
  const double S = sub_sum(rr, bps, d);
  const bool ok = active[d] != 0 && S > 0.0;
  const double v = ok ? S / rho[d] : 0.0;
  if (first_blk && threadIdx.x == 0) {
    beta[d] = v;
    rho_next[d] = ok ? S : rho[d];
    if (!ok) active[d] = 0;
  }
  return v;
}

// v = field[i] + coef x; v may be x.  A scaled format's value is its stored
// number times its scale, and that product is the one that joins the addition
// in the fused multiply-add; for FP16 component SWAP has them the other way
// round.  All of it is written out because 16-bit storage turns one rounding
// into another stored value, and the updates that were kernels of their own
// had this rounding (SWAP is what their compilation chose).  Either order is as
// exact: without SWAP the preconditioner (16^3x32 x 12, FP16, k = 6) is 6.4e-4
// from its value in 64 bits, as with it, but 3.0e-4 from what it returned
// before, so the rounding stays; tests/test_gpu_inner_rounding.py holds it.
template <int SWAP, typename S, typename T>
__device__ __forceinline__ void load_site_add(const Field<S>& f, uint32_t i, T coef, const T* x, T* v) {
  T t[24];
  if constexpr (StoreTraits<S>::scaled) {
    const T sc = load_site_unscaled(f, i, t);
#pragma unroll
    for (int k = 0; k < 24; ++k)
      v[k] = std::is_same<S, __half>::value && k == SWAP ? fmadd(coef, x[k], sc * t[k])
                                                         : fmadd(sc, t[k], coef * x[k]);
  } else {
    load_site(f, i, t);
#pragma unroll
    for (int k = 0; k < 24; ++k) v[k] = fmadd(coef, x[k], t[k]);
  }
}

// r_out = r_in - alpha q (the first step writes its residual to another buffer:
// r_in stays as its search direction)
template <typename I>
__global__ void __launch_bounds__(256)
k_sub_update(Field<I> rin, Field<I> rout, Field<I> qs, SubScalars sc, int nsub, SubTables tc, int Ls, int ns,
             const double* pq, const double* rr0, double* partial, const int* mask) {
  using T = calc_t<I>;
  __shared__ double red[16];
  const int rhs = blockIdx.y;
  if (mask && mask[rhs] == 0) return;
  rin = rin.at(rhs);
  rout = rout.at(rhs);
  qs = qs.at(rhs);
  const int64_t so = (int64_t)rhs * nsub;
  partial += (int64_t)rhs * gridDim.x;
  const CSite c = c_site(tc, ns, Ls);
  const double alpha_d = fused_alpha(pq + so * tc.bps, rr0 ? rr0 + so * tc.bps : nullptr, tc.bps, c.d,
                                     c.blk == c.d * tc.bps, sc.rho + so, sc.alpha + so, sc.active + so);
  double loc = 0;
  if (c.valid) {
    const T a = (T)alpha_d;
    T r[24], q[24];
    load_site(qs, c.in5, q);
    load_site_add<6>(rin, c.in5, -a, q, r);
#pragma unroll
    for (int k = 0; k < 24; ++k) loc += (double)r[k] * (double)r[k];
    store_site(rout, c.in5, r);
  }
  const double tot = block_sum(loc, red);
  if (threadIdx.x == 0) partial[c.blk] = tot;
}

// z (+)= alpha p, p = r + beta p, t0 = E p.  The solution's update belongs to
// the step before; it is made here, where p is read anyway (with the residual's
// update it would read p once more).
template <typename I>
__global__ void __launch_bounds__(256)
k_sub_xpay5(Field<I> ps, Field<I> rs, Field<I> zs, Field<I> t0, SubScalars sc, const double* rr, int nsub, int first,
            const calc_t<I>* E, SubTables tc, int Ls, int ns, const int* mask) {
  using T = calc_t<I>;
  const int rhs = blockIdx.y;
  if (mask && mask[rhs] == 0) return;
  ps = ps.at(rhs);
  rs = rs.at(rhs);
  zs = zs.at(rhs);
  t0 = t0.at(rhs);
  const int64_t so = (int64_t)rhs * nsub;
  extern __shared__ __align__(16) unsigned char lds_raw[];
  double* red = reinterpret_cast<double*>(lds_raw);
  T* mats = reinterpret_cast<T*>(red + 16);
  T* tile = mats + 2 * Ls * Ls;
  const CSite c = c_site(tc, ns, Ls);
  for (int k = threadIdx.x; k < 2 * Ls * Ls; k += blockDim.x) mats[k] = E[k];
  const double beta_d = fused_beta(rr + so * tc.bps, tc.bps, c.d, c.blk == c.d * tc.bps, sc.rho + so, sc.rho_next + so,
                                   sc.beta + so, sc.active + so);
  T p[24];
  if (c.valid) {
    const T a = (T)sc.alpha[so + c.d], b = (T)beta_d;
    T z[24];
    load_site(ps, c.in5, p);
    if (first) {
#pragma unroll
      for (int k = 0; k < 24; ++k) z[k] = a * p[k];
    } else {
      load_site_add<-1>(zs, c.in5, a, p, z);
    }
    store_site(zs, c.in5, z);
    load_site_add<23>(rs, c.in5, b, p, p);
    store_site(ps, c.in5, p);
  } else {
#pragma unroll
    for (int k = 0; k < 24; ++k) p[k] = 0;
  }
  T* my = tile + c.sl * tile_stride(Ls);
  if (c.inb) tile_put(my, c.s, p);
  __syncthreads();
  if (c.inb) mat5_lds(my, mats, c.s, Ls, p, false);
  if (c.valid) store_site(t0, c.in5, p);
}

// v as a field of storage S holds it: the arithmetic of store_site and load_site
template <typename S, typename T> __device__ __forceinline__ void as_stored(T* v) {
  if constexpr (StoreTraits<S>::scaled) {
    float mx = 0.f, tmp[24];
#pragma unroll
    for (int k = 0; k < 24; ++k) mx = fmaxf(mx, fabsf((float)v[k]));
    if constexpr (std::is_same<S, int8_t>::value) {
      const float inv = mx > 0.f ? 127.0f / mx : 0.f, sc = mx * (1.0f / 127.0f);
#pragma unroll
      for (int k = 0; k < 24; ++k) tmp[k] = (float)v[k] * inv;
#pragma unroll
      for (int k = 0; k < 3; ++k) {
        const uint2 q = pack8_i8(tmp + 8 * k);
        unpack8_i8(q, tmp + 8 * k);
      }
#pragma unroll
      for (int k = 0; k < 24; ++k) v[k] = tmp[k] * sc;
    } else {
      const float inv = mx > 0.f ? 1.0f / mx : 0.f;
#pragma unroll
      for (int k = 0; k < 24; ++k) tmp[k] = (float)v[k] * inv;
#pragma unroll
      for (int k = 0; k < 3; ++k) {
        const uint4 q = pack8<S>(tmp + 8 * k);
        unpack8<S>(q, tmp + 8 * k);
      }
#pragma unroll
      for (int k = 0; k < 24; ++k) v[k] = tmp[k] * mx;
    }
  }
}

// What the prolongation does to the inner solution first (pq set): the last
// step's z (+)= alpha p, rounded to the inner storage as a store would.
struct LastStep {
  const double* pq;    // partials of <p, q>; null: zs is the solution
  const double* rr0;   // partials of |r_s|^2 when there was one step only
  int nsub, first;     // first: z = alpha p
};

// z = sum_s R_s^T z_s, with the partials of <z, r> and <z, r_old> when partial1
// (partial2) is set
template <typename O, typename I>
__global__ void __launch_bounds__(256)
k_sub_prolong(Field<O> z, Field<I> zs, Field<I> ps, LastStep ls, SubScalars sc, Field<O> r, Field<O> rold, Lattice lat,
              SubTables tc, int Ls, int ns, double* partial1, double* partial2, const int* mask) {
  using T = calc_t<O>;
  using TI = calc_t<I>;
  __shared__ double red[16];
  const int rhs = blockIdx.y;
  if (mask && mask[rhs] == 0) return;
  z = z.at(rhs);
  zs = zs.at(rhs);
  ps = ps.at(rhs);
  r = r.at(rhs);
  rold = rold.at(rhs);
  const CSite c = c_site(tc, ns, Ls);
  TI a = 0;
  if (ls.pq) {
    const int64_t so = (int64_t)rhs * ls.nsub;
    a = (TI)fused_alpha(ls.pq + so * tc.bps, ls.rr0 ? ls.rr0 + so * tc.bps : nullptr, tc.bps, c.d,
                        c.blk == c.d * tc.bps, sc.rho + so, sc.alpha + so, sc.active + so);
  }
  double l1 = 0, l2 = 0;
  if (c.valid) {
    const int64_t g5 = c_global(tc, lat, c.d, c.j) * Ls + c.s;
    TI w[24];
    if (ls.pq) {
      TI p[24];
      load_site(ps, c.in5, p);
      if (ls.first) {
#pragma unroll
        for (int k = 0; k < 24; ++k) w[k] = a * p[k];
      } else {
        load_site_add<-1>(zs, c.in5, a, p, w);
      }
      as_stored<I>(w);
    } else {
      load_site(zs, c.in5, w);
    }
    T v[24], rv[24];   // z in the outer precision, as stored
#pragma unroll
    for (int k = 0; k < 24; ++k) v[k] = (T)w[k];
    store_site(z, g5, v);
    if (partial1) {
      load_site(r, g5, rv);
#pragma unroll
      for (int k = 0; k < 24; ++k) l1 += (double)v[k] * (double)rv[k];
    }
    if (partial2) {
      load_site(rold, g5, rv);
#pragma unroll
      for (int k = 0; k < 24; ++k) l2 += (double)v[k] * (double)rv[k];
    }
  }
  if (partial1) {
    const double t1 = block_sum(l1, red);
    if (threadIdx.x == 0) partial1[(int64_t)rhs * gridDim.x + c.blk] = t1;
  }
  if (partial2) {
    const double t2 = block_sum(l2, red);
    if (threadIdx.x == 0) partial2[(int64_t)rhs * gridDim.x + c.blk] = t2;
  }
}

// ---------------------------------------------------------------- launchers

static int c_ns(int Ls, Prec p) { return sites_per_block(Ls, p); }

static dim3 c_grid(int nsub, const SubTables& tc, const Batch& bt) {
  return dim3((unsigned)((int64_t)nsub * tc.bps), (unsigned)bt.n);
}

template <typename O, typename I>
static void restrict_t(hipStream_t st, const FieldPtr& r, const FieldPtr& rs, const FieldPtr& t0, const void* E,
                       const Lattice& lat, const SubTables& tc, int nsub, int Ls, double* partial,
                       const Batch& bt) {
  using T = calc_t<I>;
  const int ns = c_ns(Ls, rs.prec);
  const size_t lds = 16 * sizeof(double) + sizeof(T) * (size_t)(2 * Ls * Ls + ns * tile_stride(Ls));
  hipLaunchKernelGGL((k_sub_restrict<O, I>), c_grid(nsub, tc, bt), dim3(site_block_threads(ns, Ls)), lds, st,
                     typed<O>(r), typed<I>(rs), typed<I>(t0), (const T*)E, lat, tc, Ls, ns, partial,
                     bt.mask);
  LAUNCH_CHECK();
}

template <typename O>
static void restrict_o(hipStream_t st, Prec inner, const FieldPtr& r, const FieldPtr& rs, const FieldPtr& t0,
                       const void* E, const Lattice& lat, const SubTables& tc, int nsub, int Ls,
                       double* partial, const Batch& bt) {
  switch (inner) {
    case Prec::F64: restrict_t<O, double>(st, r, rs, t0, E, lat, tc, nsub, Ls, partial, bt); break;
    case Prec::F32: restrict_t<O, float>(st, r, rs, t0, E, lat, tc, nsub, Ls, partial, bt); break;
    case Prec::F16: restrict_t<O, __half>(st, r, rs, t0, E, lat, tc, nsub, Ls, partial, bt); break;
    case Prec::BF16: restrict_t<O, __hip_bfloat16>(st, r, rs, t0, E, lat, tc, nsub, Ls, partial, bt); break;
    case Prec::I8: restrict_t<O, int8_t>(st, r, rs, t0, E, lat, tc, nsub, Ls, partial, bt); break;
  }
}

void sub_restrict(hipStream_t st, Prec outer, Prec inner, const FieldPtr& r_outer, const FieldPtr& rs,
                  const FieldPtr& t0, const void* E, const Lattice& lat, const SubTables& tc, int nsub, int Ls,
                  double* partial, const Batch& bt) {
  if (outer == Prec::F64) restrict_o<double>(st, inner, r_outer, rs, t0, E, lat, tc, nsub, Ls, partial, bt);
  else if (outer == Prec::F32) restrict_o<float>(st, inner, r_outer, rs, t0, E, lat, tc, nsub, Ls, partial, bt);
  else throw std::runtime_error("sub_restrict: outer precision must be FP64 or FP32");
}

template <typename I>
static void update_t(hipStream_t st, const FieldPtr& rin, const FieldPtr& rout, const FieldPtr& qs,
                     const SubScalars& sc, const SubTables& tc, int nsub, int Ls, const double* pq, const double* rr0,
                     double* partial, const Batch& bt) {
  const int ns = c_ns(Ls, rin.prec);
  hipLaunchKernelGGL((k_sub_update<I>), c_grid(nsub, tc, bt), dim3(site_block_threads(ns, Ls)), 0, st, typed<I>(rin),
                     typed<I>(rout), typed<I>(qs), sc, nsub, tc, Ls, ns, pq, rr0, partial, bt.mask);
  LAUNCH_CHECK();
}

void sub_update(hipStream_t st, Prec inner, const FieldPtr& rin, const FieldPtr& rout, const FieldPtr& qs,
                const SubScalars& sc, const SubTables& tc, int nsub, int Ls, const double* pq, const double* rr0,
                double* partial, const Batch& bt) {
  switch (inner) {
    case Prec::F64: update_t<double>(st, rin, rout, qs, sc, tc, nsub, Ls, pq, rr0, partial, bt); break;
    case Prec::F32: update_t<float>(st, rin, rout, qs, sc, tc, nsub, Ls, pq, rr0, partial, bt); break;
    case Prec::F16: update_t<__half>(st, rin, rout, qs, sc, tc, nsub, Ls, pq, rr0, partial, bt); break;
    case Prec::BF16: update_t<__hip_bfloat16>(st, rin, rout, qs, sc, tc, nsub, Ls, pq, rr0, partial, bt); break;
    case Prec::I8: update_t<int8_t>(st, rin, rout, qs, sc, tc, nsub, Ls, pq, rr0, partial, bt); break;
  }
}

template <typename I>
static void xpay5_t(hipStream_t st, const FieldPtr& ps, const FieldPtr& rs, const FieldPtr& zs, const FieldPtr& t0,
                    const SubScalars& sc, const double* rr, bool first, const void* E, const SubTables& tc, int nsub,
                    int Ls, const Batch& bt) {
  using T = calc_t<I>;
  const int ns = c_ns(Ls, ps.prec);
  const size_t lds = 16 * sizeof(double) + sizeof(T) * (size_t)(2 * Ls * Ls + ns * tile_stride(Ls));
  hipLaunchKernelGGL((k_sub_xpay5<I>), c_grid(nsub, tc, bt), dim3(site_block_threads(ns, Ls)), lds, st, typed<I>(ps),
                     typed<I>(rs), typed<I>(zs), typed<I>(t0), sc, rr, nsub, first ? 1 : 0, (const T*)E, tc, Ls, ns,
                     bt.mask);
  LAUNCH_CHECK();
}

void sub_xpay5(hipStream_t st, Prec inner, const FieldPtr& ps, const FieldPtr& rs, const FieldPtr& zs,
               const FieldPtr& t0, const SubScalars& sc, const double* rr, bool first, const void* E,
               const SubTables& tc, int nsub, int Ls, const Batch& bt) {
  switch (inner) {
    case Prec::F64: xpay5_t<double>(st, ps, rs, zs, t0, sc, rr, first, E, tc, nsub, Ls, bt); break;
    case Prec::F32: xpay5_t<float>(st, ps, rs, zs, t0, sc, rr, first, E, tc, nsub, Ls, bt); break;
    case Prec::F16: xpay5_t<__half>(st, ps, rs, zs, t0, sc, rr, first, E, tc, nsub, Ls, bt); break;
    case Prec::BF16: xpay5_t<__hip_bfloat16>(st, ps, rs, zs, t0, sc, rr, first, E, tc, nsub, Ls, bt); break;
    case Prec::I8: xpay5_t<int8_t>(st, ps, rs, zs, t0, sc, rr, first, E, tc, nsub, Ls, bt); break;
  }
}

template <typename O, typename I>
static void prolong_t(hipStream_t st, const FieldPtr& z, const FieldPtr& zs, const SubLast* last, const FieldPtr& r,
                      const FieldPtr* rold, const Lattice& lat, const SubTables& tc, int nsub, int Ls, double* p1,
                      double* p2, const Batch& bt) {
  const int ns = c_ns(Ls, zs.prec);
  Field<O> ro = rold ? typed<O>(*rold) : Field<O>{};
  LastStep ls{nullptr, nullptr, nsub, 0};
  Field<I> ps{};
  SubScalars sc{};
  if (last) {
    ls.pq = last->pq;
    ls.rr0 = last->rr0;
    ls.first = last->rr0 ? 1 : 0;
    ps = typed<I>(last->ps);
    sc = last->sc;
  }
  hipLaunchKernelGGL((k_sub_prolong<O, I>), c_grid(nsub, tc, bt), dim3(site_block_threads(ns, Ls)), 0, st,
                     typed<O>(z), typed<I>(zs), ps, ls, sc, typed<O>(r), ro, lat, tc, Ls, ns, p1,
                     rold ? p2 : nullptr, bt.mask);
  LAUNCH_CHECK();
}

template <typename O>
static void prolong_o(hipStream_t st, Prec inner, const FieldPtr& z, const FieldPtr& zs, const SubLast* last,
                      const FieldPtr& r, const FieldPtr* rold, const Lattice& lat, const SubTables& tc, int nsub,
                      int Ls, double* p1, double* p2, const Batch& bt) {
  switch (inner) {
    case Prec::F64: prolong_t<O, double>(st, z, zs, last, r, rold, lat, tc, nsub, Ls, p1, p2, bt); break;
    case Prec::F32: prolong_t<O, float>(st, z, zs, last, r, rold, lat, tc, nsub, Ls, p1, p2, bt); break;
    case Prec::F16: prolong_t<O, __half>(st, z, zs, last, r, rold, lat, tc, nsub, Ls, p1, p2, bt); break;
    case Prec::BF16: prolong_t<O, __hip_bfloat16>(st, z, zs, last, r, rold, lat, tc, nsub, Ls, p1, p2, bt); break;
    case Prec::I8: prolong_t<O, int8_t>(st, z, zs, last, r, rold, lat, tc, nsub, Ls, p1, p2, bt); break;
  }
}

void sub_prolong(hipStream_t st, Prec outer, Prec inner, const FieldPtr& z_outer, const FieldPtr& zs,
                 const SubLast* last, const FieldPtr& r_outer, const FieldPtr* rold_outer, const Lattice& lat,
                 const SubTables& tc, int nsub, int Ls, double* partial1, double* partial2, const Batch& bt) {
  if (outer == Prec::F64) prolong_o<double>(st, inner, z_outer, zs, last, r_outer, rold_outer, lat, tc, nsub, Ls,
                                            partial1, partial2, bt);
  else if (outer == Prec::F32) prolong_o<float>(st, inner, z_outer, zs, last, r_outer, rold_outer, lat, tc, nsub, Ls,
                                                partial1, partial2, bt);
  else throw std::runtime_error("sub_prolong: outer precision must be FP64 or FP32");
}

}  // namespace mspcg
