// Full-lattice kernels: the hop operator with its fused epilogue, the
// fifth-dimension-only operator, layout conversions, the outer solver's
// BLAS-1 and deterministic reductions.
#include <atomic>
#include <map>
#include <mutex>
#include <stdexcept>
#include <string>

#include "kernels.h"
#include "sitekern.h"
#include "wavekern.h"

namespace mspcg {

#define LAUNCH_CHECK()                                                                \
  do {                                                                                \
    hipError_t e_ = hipGetLastError();                                                \
    if (e_ != hipSuccess) throw std::runtime_error(std::string("kernel launch: ") +   \
                                                   hipGetErrorString(e_));            \
  } while (0)

// process-wide choice of the fifth-dimension epilogue engine for FP32 and
// 16-bit site kernels with Ls <= 16: MFMA (default) or the vector ALUs
static std::atomic<int> g_mfma_epilogue{1};
void set_mfma_epilogue(bool on) { g_mfma_epilogue.store(on ? 1 : 0); }
bool mfma_epilogue() { return g_mfma_epilogue.load() != 0; }

// ---------------------------------------------------------------- static workspace
// Device memory for the entry point that allocates nothing
// (mspcg_apply_device_noalloc): every workspace that call needs is carved
// from this array.  Each device that loads the library holds its own copy
// until the process ends.  Host code never passes the array's name to a
// kernel or a copy (on the host it is a stand-in, not a device address):
// scratch_device_ptr resolves the address on each device once and the
// library uses only that pointer.
static __device__ __align__(256) unsigned char scratch[kScratchBytes];

void* scratch_device_ptr() {
  static std::mutex mu;
  static std::map<int, void*> ptr;   // device -> address of its copy
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess) throw std::runtime_error("scratch: hipGetDevice failed");
  std::lock_guard<std::mutex> lk(mu);
  auto it = ptr.find(dev);
  if (it != ptr.end()) return it->second;
  void* p = nullptr;
  const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
  if (e != hipSuccess || p == nullptr)
    throw std::runtime_error(std::string("scratch: hipGetSymbolAddress failed: ") + hipGetErrorString(e));
  ptr[dev] = p;
  return p;
}

bool uses_mfma(int Ls, Prec p) { return p != Prec::F64 && Ls <= 16 && mfma_epilogue(); }

int sites_per_block(int Ls, Prec p) {
  if (uses_mfma(Ls, p)) return 16;
  // blocks of <= 256 threads; FP64 tiles kept small for occupancy; the LDS
  // of the widest site kernel (two tiles and the matrices) stays <= 60 KB
  int ns = 256 / Ls;
  if (p == Prec::F64 && ns > 8) ns = 8;
  const size_t elem = p == Prec::F64 ? 8 : 4;
  while (ns > 1 && 128 + elem * (size_t)(6 * Ls * Ls + 2 * ns * tile_stride(Ls)) > 60 * 1024) --ns;
  if (ns < 1) ns = 1;
  return ns;
}

int64_t full_blocks(int64_t vh, int Ls, Prec p) {
  const int ns = sites_per_block(Ls, p);
  return (vh + ns - 1) / ns;
}

// ---------------------------------------------------------------- hop launch

// work items of a hop launch with nblk site blocks per RHS
static HopWork hop_work(int64_t nblk, const Batch& bt, const Sched& sc) {
  HopWork wk;
  wk.nblk = nblk;
  wk.nrhs = bt.n;
  wk.order = sc.order;
  wk.xcd = sc.xcd;
  wk.mask = bt.mask;
  wk.fdiv = make_fastdiv((uint32_t)(sc.order == 0 ? nblk : bt.n));
  return wk;
}

// The wavefront-per-16-sites kernel serves subdomain hops with Ls a multiple
// of 4 (up to 16) in FP32, FP16 and INT8 storage, where the MFMA epilogue is
// on: the non-adjoint hops h1 and h2, whose output regions grow past their
// input so that many sites lack some of the eight terms, and the 8-bit
// format's adjoint ones.  In FP16 and FP32 h3 and h4 every site has all eight
// terms and the general kernel's three or four wavefronts per 16 sites keep
// more of the neighbours in L1.  Measured per launch, us, general kernel ->
// this one:
//   FP16, Ls 12: 16^3x32, 4^3x8, h1 81 -> 74, h2 211 -> 160 (h3 122 -> 132,
//     h4 69 -> 69); 32^3x64, 8^3x16, h1 951 -> 847, h2 1867 -> 1542 (h3 1157 ->
//     1222, h4 848 -> 899)
//   INT8, Ls 16: 16^4, 4^4, h1 59 -> 47, h2 160 -> 96, h3 67 -> 63, h4 44 -> 34
//   FP32 h2: 8^4, 4^4, Ls 4 17.2 -> 11.2, Ls 8 18.2 -> 15.8, Ls 12 20.7 -> 20.2,
//     Ls 16 27.7 -> 24.4; 24^3x48, 6^3x12, 649 -> 426, 1112 -> 850, 1406 -> 1264,
//     2109 -> 1599
// Exceptions, where its one wavefront, with Ls / 4 slices of a site in series in
// each lane, is the longer chain or keeps too few neighbours in L1:
//   FP32 h1 with Ls 12 and 16: 8^4 13.5 -> 17.0 and 14.9 -> 20.2, 16^4 82 -> 85 and
//     100 -> 105, 24^3x48 603 -> 646 and 754 -> 789
//   FP32 h1 with Ls 8 but for launches of 1025 to 16384 blocks of 16 sites; at so
//     many blocks: 12.8 -> 13.1 at 384, 14.2 -> 14.8 at 704, 15.0 -> 15.1 at 768,
//     17.5 -> 17.0 at 1088, 26.9 -> 24.7 at 2560, 58.4 -> 57.7 at 6520, 105.9 ->
//     104.7 at 11264, 190 -> 203 at 18016, 289 -> 302 at 31232, 413 -> 433 at 45056
//     (Ls 4: 12.5 -> 10.3 at 384, 263 -> 239 at 45056)
//   INT8 with Ls 12 in launches of up to 1024 blocks (one such wavefront per
//     SIMD; h3, which has no centre field, 512; h2 gains at every size); at so
//     many blocks: h1 11.5 -> 12.9 at 384, 12.7 -> 14.0 at 544, 13.0 -> 13.2 at
//     704, 25.0 -> 22.6 at 2560; h3 11.6 -> 12.7 at 384, 13.7 -> 12.9 at 544, 14.2
//     -> 13.7 at 704; h4 13.3 -> 15.8 at 128, 13.8 -> 16.3 at 256, 18.7 -> 18.5 at
//     656, 21.5 -> 23.5 at 1024, 28.8 -> 25.2 at 1440
template <typename Geo, typename S> struct WaveHops {
  static constexpr bool any = false;
};
template <> struct WaveHops<SubGeo<float, float>, float> { static constexpr bool any = true; };
template <> struct WaveHops<SubGeo<float, __half, true>, __half> { static constexpr bool any = true; };
template <> struct WaveHops<SubGeo<float, __half, true>, int8_t> { static constexpr bool any = true; };

template <typename S> constexpr bool wave_takes(int Ls, bool dagger, bool has_w, int64_t nblk) {
  if (Ls % 4 != 0) return false;
  if (std::is_same<S, float>::value)
    return !dagger && (has_w || Ls == 4 || (Ls == 8 && nblk > 1024 && nblk <= 16384));
  if (std::is_same<S, __half>::value) return !dagger;
  if (Ls == 12 && (dagger || !has_w)) return nblk > (dagger && !has_w ? 512 : 1024);
  return true;
}

// The lane-per-5D-site kernel serves the 16- and 8-bit formats' subdomain hops
// with Ls 4, 8 or 16 before both: launches of up to 3072 wavefronts (three per
// SIMD), where the time is one wavefront's chain, and at every size those hops
// that its epilogue without redistribution makes faster.  Measured per launch,
// us, the other kernels -> this one, with the launch's wavefronts:
//   FP16, 4^4 and 6^4 subdomains: Ls 8 h4 256 13.0 -> 8.9, h1 768 9.6 -> 8.7, h2
//     1664 12.1 -> 9.9, 3328 15.6 -> 15.6, 5632 19.2 -> 21.3; Ls 16 h1 1536 12.6 ->
//     9.6, h4 2624 20.9 -> 17.9, h2 3328 16.2 -> 15.7, h1 6080 18.9 -> 21.9, h3
//     6080 23.7 -> 22.6
//   FP16 h4: 16^4 x 16, 4^4 52.8 -> 40.4; 24^3x48 x 4, 6^3x12 137 -> 117;
//     32^3x64 x 8, 8^3x16 623 -> 579, x 16 1196 -> 1129
//   FP16 h3: 24^3x48 x 4 199 -> 192, x 8 314 -> 295; 32^3x64 x 8 825 -> 806
//     (x 16 1432 -> 1603)
//   INT8, 24^3x48 x 4: h1 127 -> 111, h2 242 -> 211, h3 169 -> 146, h4 126 -> 100;
//     x 8: h3 248 -> 225 (h1 178 -> 186, h2 351 -> 371, h4 164 -> 168)
// In the rest the link that the wavefront kernel loads once per Ls / 4 slices,
// or the general kernel's reuse of neighbours in L1, weighs more.  Where that
// begins differs between types and Ls, and one bound for all of them refuses
// some launches that this kernel does faster: INT8 Ls 16 h1 6080 21.7 -> 18.3,
// h2 11264 34.3 -> 31.0, h3 6080 24.7 -> 21.4; INT8 Ls 8 h1 12288 33.3 -> 30.4, h4
// 4096 28.5 -> 24.6; FP16 Ls 4 h1 6144 22.3 -> 20.1, h2 13312 43.2 -> 39.4.
template <typename S> constexpr bool lane_takes(int Ls, bool dagger, bool has_w, int64_t nblk) {
  if (Ls != 4 && Ls != 8 && Ls != 16) return false;
  if (nblk * (Ls / 4) <= 3072) return true;
  if (std::is_same<S, int8_t>::value) return Ls == 4 || (Ls == 8 && dagger && !has_w);
  return dagger && (has_w || Ls <= 8);
}

enum class SubHop { General, Wave, Lane };
template <typename S> constexpr SubHop sub_hop(int Ls, bool dagger, bool has_w, int64_t nblk) {
  if (sizeof(S) < 4 && lane_takes<S>(Ls, dagger, has_w, nblk)) return SubHop::Lane;
  return wave_takes<S>(Ls, dagger, has_w, nblk) ? SubHop::Wave : SubHop::General;
}

// the instances there are: those that sub_hop reaches (the lane kernel: all of
// Ls 4, 8 and 16)
template <typename S> constexpr bool has_wave(int Ls, bool dagger, bool has_w) {
  if (std::is_same<S, float>::value) return !dagger && (has_w || Ls <= 8);
  if (std::is_same<S, __half>::value) return !dagger;
  return Ls > 8 || (Ls == 8 && (!dagger || has_w));
}
template <typename S> constexpr bool has_general(bool dagger, bool has_w) {
  if (std::is_same<S, float>::value) return true;
  return dagger || (std::is_same<S, int8_t>::value && !has_w);
}

// no launch that sub_hop can make, on either side of each of its bounds, lacks its kernel
template <typename S> constexpr bool hops_have_kernels() {
  constexpr int64_t n[] = {1, 192, 193, 512, 513, 768, 769, 1024, 1025, 1536, 1537, 3072, 3073, 16384, 16385, 1 << 30};
  for (int Ls = 4; Ls <= 16; Ls += 4)
    for (int64_t nblk : n)
      for (int f = 0; f < 4; ++f) {
        const SubHop k = sub_hop<S>(Ls, f & 1, f & 2, nblk);
        if (k == SubHop::Wave && !has_wave<S>(Ls, f & 1, f & 2)) return false;
        if (k == SubHop::General && !has_general<S>(f & 1, f & 2)) return false;
      }
  return true;
}
static_assert(hops_have_kernels<float>() && hops_have_kernels<__half>() && hops_have_kernels<int8_t>(),
              "a subdomain hop's kernel is not instantiated");

template <typename F> static void by_flag(bool v, F&& f) {
  if (v) f(std::true_type());
  else f(std::false_type());
}
template <typename F> static void by_ls(int Ls, F&& f) {
  switch (Ls) {
    case 4: f(std::integral_constant<int, 4>()); break;
    case 8: f(std::integral_constant<int, 8>()); break;
    case 12: f(std::integral_constant<int, 12>()); break;
    case 16: f(std::integral_constant<int, 16>()); break;
    default: throw std::runtime_error("hop: Ls is no multiple of 4 up to 16");
  }
}

template <typename Geo, typename S, bool MF>
static void launch_hop_mf(hipStream_t st, const Geo& geo, int64_t nblocks, const FieldPtr& out, const FieldPtr& in,
                          const FieldPtr* w, int Ls, int ns, bool dagger, const Epilogue& epi, const Batch& bt,
                          const Sched& sc) {
  using T = calc_t<S>;
  if (epi.dot_partial && !(dagger && w))
    throw std::runtime_error("hop: the fused dot belongs to an adjoint hop with a centre field");
  const bool tileB = w != nullptr && !epi.w_identity && epi.E0 != nullptr;
  const size_t lds = site_lds_bytes<T>(ns, Ls, tileB, MF, UsesMfma<S>::half_ops);
  Field<S> wf = w ? typed<S>(*w) : Field<S>{};
  Field<S> df = epi.dotf ? typed<S>(*epi.dotf) : Field<S>{};
  const T* E0 = (const T*)epi.E0;
  const T* E1 = (const T*)epi.E1;
  const HopWork wk = hop_work(nblocks, bt, sc);
  dim3 grid((unsigned)(nblocks * bt.n)), block(site_block_threads(ns, Ls));
  const int wid = epi.w_identity ? 1 : 0;
  if constexpr (MF && WaveHops<Geo, S>::any) {
    const SubHop kernel = E1 && (!w || tileB) ? sub_hop<S>(Ls, dagger, w != nullptr, nblocks * bt.n) : SubHop::General;
    if (kernel != SubHop::General) {
      by_ls(Ls, [&](auto ls) {
        by_flag(dagger, [&](auto dag) {
          by_flag(w != nullptr, [&](auto hw) {
            constexpr int L = decltype(ls)::value;
            constexpr bool D = decltype(dag)::value, W = decltype(hw)::value;
            if (kernel == SubHop::Lane) {
              if constexpr (sizeof(S) < 4 && L != 12)
                hipLaunchKernelGGL((k_hop_lane<Geo, S, L, D, W>), grid, dim3(16 * L), 0, st, geo, typed<S>(out),
                                   typed<S>(in), wf, df, E0, E1, epi.dot_partial, wk);
              else throw std::runtime_error("hop: no lane kernel for this storage and Ls");
            } else {
              if constexpr (has_wave<S>(L, D, W))
                hipLaunchKernelGGL((k_hop_wave<Geo, S, L / 4, D, W>), grid, dim3(64), 0, st, geo, typed<S>(out),
                                   typed<S>(in), wf, df, E0, E1, epi.dot_partial, wk);
              else throw std::runtime_error("hop: no wavefront kernel for this storage, Ls and hop");
            }
          });
        });
      });
      LAUNCH_CHECK();
      return;
    }
  }
  by_flag(dagger, [&](auto dag) {
    by_flag(w != nullptr, [&](auto hw) {
      constexpr bool D = decltype(dag)::value, W = decltype(hw)::value;
      if constexpr (!(MF && WaveHops<Geo, S>::any) || has_general<S>(D, W))
        hipLaunchKernelGGL((k_hop<Geo, S, D, W, MF>), grid, block, lds, st, geo, typed<S>(out), typed<S>(in), wf, df, Ls,
                           ns, E0, E1, wid, epi.dot_partial, wk);
      else throw std::runtime_error("hop: no general kernel for this storage and hop");
    });
  });
  LAUNCH_CHECK();
}

template <typename Geo, typename S>
static void launch_hop(hipStream_t st, const Geo& geo, int64_t nblocks, const FieldPtr& out, const FieldPtr& in,
                       const FieldPtr* w, int Ls, int ns, bool dagger, const Epilogue& epi, const Batch& bt,
                       const Sched& sc) {
  if (bt.n < 1) throw std::runtime_error("hop: batch of fewer than one RHS");
  if constexpr (std::is_same<S, double>::value) {
    launch_hop_mf<Geo, S, false>(st, geo, nblocks, out, in, w, Ls, ns, dagger, epi, bt, sc);
  } else {
    if (uses_mfma(Ls, out.prec)) launch_hop_mf<Geo, S, true>(st, geo, nblocks, out, in, w, Ls, ns, dagger, epi, bt, sc);
    else launch_hop_mf<Geo, S, false>(st, geo, nblocks, out, in, w, Ls, ns, dagger, epi, bt, sc);
  }
}

int64_t hop_full_blocks(const Lattice& lat, int Ls, Prec p) {
  const int ns = sites_per_block(Ls, p);
  return (lat.vh + ns - 1) / ns;
}

// Chunk shape of the chunked block order (BlockOrder): bzc z-planes by bb
// blocks of a plane whose input spinors take at most `budget` bytes, with the
// fewest neighbour planes and rows outside the chunk per site inside it
// (2 / bzc + 2 / rows, a dimension the chunk spans whole counting 0).
// Lexicographic order when blocks do not tile whole planes.
static BlockOrder block_order(const Lattice& lat, int ns, int Ls, int site_bytes, int64_t budget) {
  BlockOrder bo{};
  bo.chunk = 0;
  const int64_t S = lat.vh / lat.T, P = (int64_t)lat.X * lat.Y / 2, half_x = lat.X / 2;
  if (lat.vh % lat.T || S % ns || P % ns) return bo;
  const int64_t bz = P / ns, blk_bytes = (int64_t)ns * Ls * site_bytes;
  double best = 1e30;
  int64_t bbz = 0, bbb = 0;
  for (int64_t zc = 1; zc <= lat.Z; ++zc) {
    if (lat.Z % zc) continue;
    for (int64_t b = 1; b <= bz; ++b) {
      if (bz % b) continue;
      if (b < bz && (b * ns) % half_x) continue;   // a band of whole rows
      if (zc * b * blk_bytes > budget) continue;
      const double halo = (zc < lat.Z ? 2.0 / zc : 0.0) + (b < bz ? 2.0 * half_x / (b * ns) : 0.0);
      if (halo < best - 1e-12 || (halo < best + 1e-12 && zc * b > bbz * bbb)) {
        best = halo;
        bbz = zc;
        bbb = b;
      }
    }
  }
  if (bbz == 0 || (bbz == lat.Z && bbb == bz)) return bo;   // whole slices: the lexicographic order
  bo.chunk = (uint32_t)(bbz * bbb);
  bo.bzc = (uint32_t)bbz;
  bo.bb = (uint32_t)bbb;
  bo.bz = (uint32_t)bz;
  bo.bps = (uint32_t)(S / ns);
  bo.fchunk = make_fastdiv(bo.chunk);
  bo.fT = make_fastdiv((uint32_t)lat.T);
  bo.fbb = make_fastdiv(bo.bb);
  bo.fnyc = make_fastdiv((uint32_t)(bz / bbb));
  return bo;
}

template <typename S>
static void hop_full_t(hipStream_t st, const FieldPtr& out, const FieldPtr& in, const FieldPtr* w, const void* gauge,
                       const HopGeometry& geo, bool dagger, const Epilogue& epi, const Batch& bt, const Sched& sc) {
  using T = calc_t<S>;
  FullGeo<T> g;
  g.lat = geo.lat;
  g.par = geo.out_parity;
  g.g.data = reinterpret_cast<const typename Gauge<T>::c2*>(gauge);
  g.g.vh = geo.lat.vh;
  const int ns = sites_per_block(geo.Ls, out.prec);
  g.order.chunk = 0;
  if (sc.tchunk > 0 && geo.lat.vh < (int64_t)1 << 31)
    g.order = block_order(geo.lat, ns, geo.Ls, 24 * (int)sizeof(T), (int64_t)80 << (10 + sc.tchunk));
  launch_hop<FullGeo<T>, S>(st, g, (geo.lat.vh + ns - 1) / ns, out, in, w, geo.Ls, ns, dagger, epi, bt, sc);
}

void hop_full(hipStream_t st, Prec p, const FieldPtr& out, const FieldPtr& in, const FieldPtr* w,
              const void* gauge, const HopGeometry& geo, bool dagger, const Epilogue& epi, const Batch& bt,
              const Sched& sc) {
  switch (p) {
    case Prec::F64: hop_full_t<double>(st, out, in, w, gauge, geo, dagger, epi, bt, sc); break;
    case Prec::F32: hop_full_t<float>(st, out, in, w, gauge, geo, dagger, epi, bt, sc); break;
    case Prec::F16: hop_full_t<__half>(st, out, in, w, gauge, geo, dagger, epi, bt, sc); break;
    case Prec::BF16: hop_full_t<__hip_bfloat16>(st, out, in, w, gauge, geo, dagger, epi, bt, sc); break;
    case Prec::I8: hop_full_t<int8_t>(st, out, in, w, gauge, geo, dagger, epi, bt, sc); break;
  }
}

template <typename S>
static void hop_sub_t(hipStream_t st, const FieldPtr& out, const FieldPtr& in, const FieldPtr* w, const void* gauge,
                      const Lattice& lat, int out_parity, const SubTables& tb, int nsub, int Ls, bool dagger,
                      const Epilogue& epi, const Batch& bt, const Sched& sc) {
  using T = calc_t<S>;
  using L = typename std::conditional<StoreTraits<S>::scaled, __half, T>::type;
  constexpr bool half = std::is_same<S, __half>::value || std::is_same<S, int8_t>::value;
  const int ns = sites_per_block(Ls, out.prec);
  // FP16 and 8-bit storage with Ls a multiple of 4: SU(3) products on 4 x 4 x 4
  // MFMA blocks (each block's four lanes are four slices of one 4D site)
  if (half && Ls % 4 == 0) {
    SubGeo<T, L, half> g;
    g.tb = tb;
    g.lat = lat;
    g.par = out_parity;
    g.g.data = reinterpret_cast<const typename Gauge<L>::c2*>(gauge);
    g.g.vh = lat.vh;
    launch_hop<SubGeo<T, L, half>, S>(st, g, (int64_t)nsub * tb.bps, out, in, w, Ls, ns, dagger, epi, bt, sc);
    return;
  }
  SubGeo<T, L> g;
  g.tb = tb;
  g.lat = lat;
  g.par = out_parity;
  g.g.data = reinterpret_cast<const typename Gauge<L>::c2*>(gauge);
  g.g.vh = lat.vh;
  launch_hop<SubGeo<T, L>, S>(st, g, (int64_t)nsub * tb.bps, out, in, w, Ls, ns, dagger, epi, bt, sc);
}

void hop_sub(hipStream_t st, Prec p, const FieldPtr& out, const FieldPtr& in, const FieldPtr* w, const void* gauge,
             const Lattice& lat, int out_parity, const SubTables& tb, int nsub, int Ls, bool dagger,
             const Epilogue& epi, const Batch& bt, const Sched& sc) {
  switch (p) {
    case Prec::F64: hop_sub_t<double>(st, out, in, w, gauge, lat, out_parity, tb, nsub, Ls, dagger, epi, bt, sc); break;
    case Prec::F32: hop_sub_t<float>(st, out, in, w, gauge, lat, out_parity, tb, nsub, Ls, dagger, epi, bt, sc); break;
    case Prec::F16: hop_sub_t<__half>(st, out, in, w, gauge, lat, out_parity, tb, nsub, Ls, dagger, epi, bt, sc); break;
    case Prec::BF16:
      hop_sub_t<__hip_bfloat16>(st, out, in, w, gauge, lat, out_parity, tb, nsub, Ls, dagger, epi, bt, sc);
      break;
    case Prec::I8: hop_sub_t<int8_t>(st, out, in, w, gauge, lat, out_parity, tb, nsub, Ls, dagger, epi, bt, sc); break;
  }
}

// ---------------------------------------------------------------- 5D-only ops

// out = E w (copy when E is null); optional |out|^2 partial per block.
// With beta_slot >= 0 the input is first updated in place,
//   w <- z + beta w  (beta = scal[beta_slot]),
// which is the search-direction update of CG fused with the M_phi that
// starts the next operator application.
template <typename S>
__global__ void __launch_bounds__(256)
k_apply5(Field<S> out, Field<S> w, Field<S> z, const double* scal, int beta_slot, int64_t nsites, int Ls, int ns,
         const calc_t<S>* E, double* norm_partial, const int* mask) {
  using T = calc_t<S>;
  const int rhs = blockIdx.y;
  if (mask && mask[rhs] == 0) return;   // uniform over the workgroup
  out = out.at(rhs);
  w = w.at(rhs);
  z = z.at(rhs);
  extern __shared__ __align__(16) unsigned char lds_raw[];
  double* red = reinterpret_cast<double*>(lds_raw);
  T* mats = reinterpret_cast<T*>(red + 16);
  T* tileA = mats + 2 * Ls * Ls;
  const int tid = threadIdx.x;
  const bool inb = tid < ns * Ls;
  const int sl = inb ? tid / Ls : 0, s = inb ? tid - sl * Ls : 0;
  const int64_t blk = xcd_block(blockIdx.x, gridDim.x);
  const int64_t site = blk * ns + sl;
  const bool valid = inb && site < nsites;
  const int64_t i5 = site * Ls + s;
  if (E)
    for (int k = tid; k < 2 * Ls * Ls; k += blockDim.x) mats[k] = E[k];
  T v[24];
  if (valid) {
    load_site(w, i5, v);
    if (beta_slot >= 0) {
      const T beta = (T)scal[(int64_t)rhs * SLOT_COUNT + beta_slot];
      T zv[24];
      load_site(z, i5, zv);
#pragma unroll
      for (int k = 0; k < 24; ++k) v[k] = zv[k] + beta * v[k];
      store_site(w, i5, v);
    }
  } else {
#pragma unroll
    for (int k = 0; k < 24; ++k) v[k] = 0;
  }
  T* my = tileA + sl * tile_stride(Ls);
  if (inb) tile_put(my, s, v);
  __syncthreads();
  if (E && inb) mat5_lds(my, mats, s, Ls, v, false);
  if (norm_partial) {
    double loc = 0;
    if (valid) {
#pragma unroll
      for (int k = 0; k < 24; ++k) loc += (double)v[k] * (double)v[k];
    }
    const double tot = block_sum(loc, red);
    if (tid == 0) norm_partial[(int64_t)rhs * gridDim.x + blk] = tot;
  }
  if (valid) store_site(out, i5, v);
}

template <typename S>
static void apply5_t(hipStream_t st, const FieldPtr& out, const FieldPtr& w, const FieldPtr* z, const double* scal,
                     int beta_slot, const void* E, int64_t nsites, int Ls, double* norm_partial, const Batch& bt) {
  using T = calc_t<S>;
  const int ns = sites_per_block(Ls, out.prec);
  const int64_t nb = (nsites + ns - 1) / ns;
  const size_t lds = 16 * sizeof(double) + sizeof(T) * (size_t)(2 * Ls * Ls + ns * tile_stride(Ls));
  Field<S> zf = z ? typed<S>(*z) : Field<S>{};
  hipLaunchKernelGGL((k_apply5<S>), dim3((unsigned)nb, (unsigned)bt.n), dim3(site_block_threads(ns, Ls)), lds, st,
                     typed<S>(out), typed<S>(w), zf, scal, beta_slot, nsites, Ls, ns, (const T*)E, norm_partial,
                     bt.mask);
  LAUNCH_CHECK();
}

void apply5_full(hipStream_t st, Prec p, const FieldPtr& out, const FieldPtr& w, const void* E, int64_t nsites,
                 int Ls, double* norm_partial, const Batch& bt) {
  switch (p) {
    case Prec::F64: apply5_t<double>(st, out, w, nullptr, nullptr, -1, E, nsites, Ls, norm_partial, bt); break;
    case Prec::F32: apply5_t<float>(st, out, w, nullptr, nullptr, -1, E, nsites, Ls, norm_partial, bt); break;
    case Prec::F16: apply5_t<__half>(st, out, w, nullptr, nullptr, -1, E, nsites, Ls, norm_partial, bt); break;
    case Prec::BF16: apply5_t<__hip_bfloat16>(st, out, w, nullptr, nullptr, -1, E, nsites, Ls, norm_partial, bt); break;
    case Prec::I8: apply5_t<int8_t>(st, out, w, nullptr, nullptr, -1, E, nsites, Ls, norm_partial, bt); break;
  }
}

void xpay_apply5(hipStream_t st, Prec p, const FieldPtr& out, const FieldPtr& pvec, const FieldPtr& z,
                 const double* scal, int beta_slot, const void* E, int64_t nsites, int Ls, const Batch& bt) {
  switch (p) {
    case Prec::F64: apply5_t<double>(st, out, pvec, &z, scal, beta_slot, E, nsites, Ls, nullptr, bt); break;
    case Prec::F32: apply5_t<float>(st, out, pvec, &z, scal, beta_slot, E, nsites, Ls, nullptr, bt); break;
    default: throw std::runtime_error("xpay_apply5: outer vectors are FP64 or FP32");
  }
}

// ---------------------------------------------------------------- layout conversion

// A workgroup converts a run of ns sites with all their slices (ns Ls <= 256
// rows of 24 reals) through LDS: the canonical side is moved as the run's Ls
// contiguous pieces of 192 ns bytes, 16 bytes a lane, the internal side as
// whole chunks of consecutive (site, s) rows.  One thread per row reading or
// writing its 192 canonical bytes by itself touched 64 cache lines per
// instruction.  Bound by HBM: 12.6 M FP32 rows (3.6 GB) unpacked in 661 us
// (5.5 TB/s; 1147 us a thread per row), packed in 714 (794).
// (CanonPair: a caller's buffer is aligned to its doubles only)
typedef double CanonPair __attribute__((ext_vector_type(2), aligned(8)));

struct RunMap {
  int ns;
  FastDiv run;   // division by 12 ns (complex numbers of one slice of the run)
};

// complex number q (0 .. 12 ns Ls - 1) of the run: its place in the canonical
// field and its row and component in the LDS tile
struct RunPlace {
  int64_t canon;   // in complex numbers
  int lds;
  bool valid;
};
__device__ __forceinline__ RunPlace run_place(const RunMap& m, uint32_t q, int64_t site0, int64_t nsites, int Ls) {
  const uint32_t s = m.run.div(q), rem = q - s * m.run.d, sl = rem / 12u, c = rem - 12u * sl;
  RunPlace r;
  r.valid = (int)s < Ls && site0 + sl < nsites;
  r.canon = ((int64_t)s * nsites + site0) * 12 + rem;
  r.lds = (int)(sl * (uint32_t)(tile_stride(Ls) / 2) + s * 12u + c);
  return r;
}

// With EPI (FP64 and FP32, whose stored values are exact): also out2 = E out,
// the fifth-dimension operator that the application of A, D or D^dag starts
// with, from the rows in LDS: 972 us for 12.6 M FP32 rows, where packing and a
// launch of that operator by itself took 794 + 437.
template <typename S, bool EPI>
__global__ void __launch_bounds__(256)
k_pack(Field<S> out, Field<S> out2, const calc_t<S>* E, const CanonPair* canon, int64_t nsites, int Ls, RunMap m,
       const int* mask) {
  using T = calc_t<S>;
  using T2 = typename std::conditional<sizeof(T) == 8, double2, float2>::type;
  extern __shared__ __align__(16) unsigned char lds_raw[];
  T2* tile = reinterpret_cast<T2*>(lds_raw);
  T* mats = reinterpret_cast<T*>(lds_raw) + m.ns * tile_stride(Ls);
  const int rhs = blockIdx.y;
  if (mask && mask[rhs] == 0) return;
  out = out.at(rhs);
  out2 = out2.at(rhs);
  canon += (int64_t)rhs * nsites * Ls * 12;
  const int tid = threadIdx.x;
  const int64_t site0 = (int64_t)blockIdx.x * m.ns;
  CanonPair v[12];
  RunPlace pl[12];
#pragma unroll
  for (int i = 0; i < 12; ++i) {
    pl[i] = run_place(m, (uint32_t)(i * 256 + tid), site0, nsites, Ls);
    v[i] = pl[i].valid ? canon[pl[i].canon] : CanonPair{0.0, 0.0};
  }
  if constexpr (EPI)
    for (int k = tid; k < 2 * Ls * Ls; k += 256) mats[k] = E[k];
#pragma unroll
  for (int i = 0; i < 12; ++i)
    if (pl[i].valid) {
      T2 c;
      c.x = (T)v[i].x;
      c.y = (T)v[i].y;
      tile[pl[i].lds] = c;
    }
  __syncthreads();
  const int64_t i5 = site0 * Ls + tid;
  if (tid < m.ns * Ls && i5 < nsites * Ls) {
    const int sl = tid / Ls, s = tid - sl * Ls;
    const T* site = reinterpret_cast<const T*>(tile) + sl * tile_stride(Ls);
    T row[24];
#pragma unroll
    for (int k = 0; k < 24; ++k) row[k] = site[s * 24 + k];
    store_site(out, (uint32_t)i5, row);
    if constexpr (EPI) {
      mat5_lds(site, mats, s, Ls, row, false);
      store_site(out2, (uint32_t)i5, row);
    }
  }
}

template <typename S>
__global__ void __launch_bounds__(256)
k_unpack(CanonPair* canon, Field<S> in, int64_t nsites, int Ls, RunMap m, const int* mask) {
  using T = calc_t<S>;
  using T2 = typename std::conditional<sizeof(T) == 8, double2, float2>::type;
  extern __shared__ __align__(16) unsigned char lds_raw[];
  T2* tile = reinterpret_cast<T2*>(lds_raw);
  const int rhs = blockIdx.y;
  if (mask && mask[rhs] == 0) return;
  in = in.at(rhs);
  canon += (int64_t)rhs * nsites * Ls * 12;
  const int tid = threadIdx.x;
  const int64_t site0 = (int64_t)blockIdx.x * m.ns, i5 = site0 * Ls + tid;
  if (tid < m.ns * Ls && i5 < nsites * Ls) {
    T row[24];
    load_site(in, (uint32_t)i5, row);
    const int sl = tid / Ls, s = tid - sl * Ls;
    tile_put(reinterpret_cast<T*>(tile) + sl * tile_stride(Ls), s, row);
  }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < 12; ++i) {
    const RunPlace pl = run_place(m, (uint32_t)(i * 256 + tid), site0, nsites, Ls);
    if (pl.valid) {
      const T2 c = tile[pl.lds];
      canon[pl.canon] = CanonPair{(double)c.x, (double)c.y};
    }
  }
}

template <typename S>
static void pack_t(hipStream_t st, const FieldPtr& out, const double* canon, int64_t nsites, int Ls, const Batch& bt,
                   const FieldPtr* out2 = nullptr, const void* E = nullptr) {
  using T = calc_t<S>;
  RunMap m;
  m.ns = 256 / Ls;
  const auto lds_bytes = [&](int ns) { return sizeof(T) * (size_t)(ns * tile_stride(Ls) + (out2 ? 2 * Ls * Ls : 0)); };
  while (m.ns > 1 && lds_bytes(m.ns) > 60 * 1024) --m.ns;   // FP64 with the matrices of Ls > 27
  m.run = make_fastdiv((uint32_t)(12 * m.ns));
  const dim3 grid((unsigned)((nsites + m.ns - 1) / m.ns), (unsigned)bt.n);
  const size_t lds = lds_bytes(m.ns);
  if constexpr (!StoreTraits<S>::scaled) {
    if (out2) {
      hipLaunchKernelGGL((k_pack<S, true>), grid, dim3(256), lds, st, typed<S>(out), typed<S>(*out2), (const T*)E,
                         (const CanonPair*)canon, nsites, Ls, m, bt.mask);
      LAUNCH_CHECK();
      return;
    }
  }
  hipLaunchKernelGGL((k_pack<S, false>), grid, dim3(256), lds, st, typed<S>(out), Field<S>{}, (const T*)nullptr,
                     (const CanonPair*)canon, nsites, Ls, m, bt.mask);
  LAUNCH_CHECK();
}

template <typename S>
static void unpack_t(hipStream_t st, double* canon, const FieldPtr& in, int64_t nsites, int Ls, const Batch& bt) {
  RunMap m;
  m.ns = 256 / Ls;
  m.run = make_fastdiv((uint32_t)(12 * m.ns));
  const dim3 grid((unsigned)((nsites + m.ns - 1) / m.ns), (unsigned)bt.n);
  hipLaunchKernelGGL(k_unpack<S>, grid, dim3(256), sizeof(calc_t<S>) * (size_t)(m.ns * tile_stride(Ls)), st, (CanonPair*)canon,
                     typed<S>(in), nsites, Ls, m, bt.mask);
  LAUNCH_CHECK();
}

void pack_field(hipStream_t st, const FieldPtr& out, const double* canon, int64_t nsites, int Ls, const Batch& bt) {
  switch (out.prec) {
    case Prec::F64: pack_t<double>(st, out, canon, nsites, Ls, bt); break;
    case Prec::F32: pack_t<float>(st, out, canon, nsites, Ls, bt); break;
    case Prec::F16: pack_t<__half>(st, out, canon, nsites, Ls, bt); break;
    case Prec::BF16: pack_t<__hip_bfloat16>(st, out, canon, nsites, Ls, bt); break;
    case Prec::I8: pack_t<int8_t>(st, out, canon, nsites, Ls, bt); break;
  }
}

void pack_apply5(hipStream_t st, const FieldPtr& out, const FieldPtr& out2, const void* E, const double* canon,
                 int64_t nsites, int Ls) {
  switch (out.prec) {
    case Prec::F64: pack_t<double>(st, out, canon, nsites, Ls, Batch(), &out2, E); break;
    case Prec::F32: pack_t<float>(st, out, canon, nsites, Ls, Batch(), &out2, E); break;
    default:   // the operator acts on the values as stored
      pack_field(st, out, canon, nsites, Ls);
      apply5_full(st, out.prec, out2, out, E, nsites, Ls, nullptr);
  }
}

void unpack_field(hipStream_t st, double* canon, const FieldPtr& in, int64_t nsites, int Ls, const Batch& bt) {
  switch (in.prec) {
    case Prec::F64: unpack_t<double>(st, canon, in, nsites, Ls, bt); break;
    case Prec::F32: unpack_t<float>(st, canon, in, nsites, Ls, bt); break;
    case Prec::F16: unpack_t<__half>(st, canon, in, nsites, Ls, bt); break;
    case Prec::BF16: unpack_t<__hip_bfloat16>(st, canon, in, nsites, Ls, bt); break;
    case Prec::I8: unpack_t<int8_t>(st, canon, in, nsites, Ls, bt); break;
  }
}

// zero every masked RHS of a batched buffer (a kernel, so that it may sit in
// a captured graph)
__global__ void k_zero(uint4* data, int64_t n16, const int* mask) {
  const int rhs = blockIdx.y;
  if (mask && mask[rhs] == 0) return;
  uint4* d = data + (int64_t)rhs * n16;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n16; i += (int64_t)gridDim.x * blockDim.x)
    d[i] = make_uint4(0u, 0u, 0u, 0u);
}

__global__ void k_fill_int(int* p, int n, int v) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = v;
}

void fill_int(hipStream_t st, int* p, int n, int v) {
  if (n <= 0) return;
  hipLaunchKernelGGL(k_fill_int, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, p, n, v);
  LAUNCH_CHECK();
}

void zero_batched(hipStream_t st, void* data, int64_t bytes_per_rhs, const Batch& bt) {
  if (bytes_per_rhs % 16) throw std::runtime_error("zero_batched: size must be a multiple of 16 bytes");
  const int64_t n16 = bytes_per_rhs / 16;
  int64_t nb = (n16 + 255) / 256;
  if (nb > 2048) nb = 2048;
  if (nb < 1) nb = 1;
  hipLaunchKernelGGL(k_zero, dim3((unsigned)nb, (unsigned)bt.n), dim3(256), 0, st, (uint4*)data, n16, bt.mask);
  LAUNCH_CHECK();
}

template <typename C2>
__global__ void k_pack_gauge(C2* out, const double* canon, Lattice lat) {
  const int64_t lex = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t V = 2 * lat.vh;
  if (lex >= V) return;
  const int x = (int)(lex % lat.X);
  const int64_t r = lex / lat.X;
  const int y = (int)(r % lat.Y);
  const int64_t r2 = r / lat.Y;
  const int z = (int)(r2 % lat.Z);
  const int t = (int)(r2 / lat.Z);
  const int par = (x + y + z + t) & 1;
  const int64_t cb = lex >> 1;
  for (int mu = 0; mu < 4; ++mu)
    for (int k = 0; k < 9; ++k) {
      const double* src = canon + ((lex * 4 + mu) * 9 + k) * 2;
      C2 c;
      if constexpr (sizeof(C2) == 4) {
        c.x = __float2half_rn((float)src[0]);
        c.y = __float2half_rn((float)src[1]);
      } else {
        c.x = src[0];
        c.y = src[1];
      }
      out[((int64_t)(par * 4 + mu) * lat.vh + cb) * 10 + k] = c;
    }
}

void pack_gauge(hipStream_t st, void* out, int bytes_per_real, const double* canon, const Lattice& lat) {
  const int64_t V = 2 * lat.vh;
  dim3 grid((unsigned)((V + 255) / 256)), block(256);
  if (bytes_per_real == 8) hipLaunchKernelGGL(k_pack_gauge<double2>, grid, block, 0, st, (double2*)out, canon, lat);
  else if (bytes_per_real == 4) hipLaunchKernelGGL(k_pack_gauge<float2>, grid, block, 0, st, (float2*)out, canon, lat);
  else hipLaunchKernelGGL(k_pack_gauge<__half2>, grid, block, 0, st, (__half2*)out, canon, lat);
  LAUNCH_CHECK();
}

// ---------------------------------------------------------------- outer BLAS-1
//
// Outer vectors (FP64 or FP32) are flat arrays of chunks; every kernel runs
// a fixed grid so its per-block partial sums land in a fixed order.

int64_t blas_blocks(int64_t nchunks) {
  int64_t nb = (nchunks + 255) / 256;
  return nb > 2048 ? 2048 : (nb < 1 ? 1 : nb);
}

template <typename C> struct ChunkOps;
template <> struct ChunkOps<float4> {
  static constexpr int n = 4;
  __device__ static float get(const float4& c, int k) { return k == 0 ? c.x : k == 1 ? c.y : k == 2 ? c.z : c.w; }
  __device__ static void set(float4& c, int k, float v) {
    if (k == 0) c.x = v; else if (k == 1) c.y = v; else if (k == 2) c.z = v; else c.w = v;
  }
};
template <> struct ChunkOps<double2> {
  static constexpr int n = 2;
  __device__ static double get(const double2& c, int k) { return k == 0 ? c.x : c.y; }
  __device__ static void set(double2& c, int k, double v) { if (k == 0) c.x = v; else c.y = v; }
};

// Batched launches put the RHS in blockIdx.y: RHS r of a vector starts r
// whole vectors after RHS 0, its scalars at scal + r * SLOT_COUNT and its
// block partials at partial + r * gridDim.x.

// x += alpha p ; rn = r - alpha q ; partial |rn|^2     (alpha = scal[alpha_slot])
template <typename C>
__global__ void __launch_bounds__(256)
k_cg_update(C* x, const C* p, const C* r, const C* q, C* rn, int64_t n, const double* scal, int alpha_slot,
            double* partial, const int* mask) {
  __shared__ double red[16];
  using O = ChunkOps<C>;
  const int rhs = blockIdx.y;
  if (mask && mask[rhs] == 0) return;
  const int64_t off = (int64_t)rhs * n;
  x += off; p += off; r += off; q += off; rn += off;
  const double alpha = scal[(int64_t)rhs * SLOT_COUNT + alpha_slot];
  double loc = 0;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
    C xv = x[i], pv = p[i], rv = r[i], qv = q[i], ov;
#pragma unroll
    for (int k = 0; k < O::n; ++k) {
      O::set(xv, k, O::get(xv, k) + alpha * O::get(pv, k));
      const double v = O::get(rv, k) - alpha * O::get(qv, k);
      O::set(ov, k, v);
      const double vs = O::get(ov, k);
      loc += vs * vs;
    }
    x[i] = xv;
    rn[i] = ov;
  }
  const double tot = block_sum(loc, red);
  if (threadIdx.x == 0) partial[(int64_t)rhs * gridDim.x + blockIdx.x] = tot;
}

// partial Re<a, b1>, Re<a, b2> (b2 nullable)
template <typename C>
__global__ void __launch_bounds__(256)
k_dot2(const C* a, const C* b1, const C* b2, int64_t n, double* partial1, double* partial2, const int* mask) {
  __shared__ double red[16];
  using O = ChunkOps<C>;
  const int rhs = blockIdx.y;
  if (mask && mask[rhs] == 0) return;
  const int64_t off = (int64_t)rhs * n;
  a += off;
  b1 += off;
  if (b2) b2 += off;
  double l1 = 0, l2 = 0;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
    const C av = a[i], bv = b1[i];
#pragma unroll
    for (int k = 0; k < O::n; ++k) l1 += (double)O::get(av, k) * (double)O::get(bv, k);
    if (b2) {
      const C cv = b2[i];
#pragma unroll
      for (int k = 0; k < O::n; ++k) l2 += (double)O::get(av, k) * (double)O::get(cv, k);
    }
  }
  const int64_t pi = (int64_t)rhs * gridDim.x + blockIdx.x;
  double t1 = block_sum(l1, red);
  if (threadIdx.x == 0) partial1[pi] = t1;
  if (b2) {
    double t2 = block_sum(l2, red);
    if (threadIdx.x == 0) partial2[pi] = t2;
  }
}

// Mixed-precision helpers.  An FP32 chunk j of 5D site i holds complex
// numbers 2j and 2j+1 of that site; in FP64 they are chunks 2j and 2j+1.
// Both layouts use stride n5 (chunks per chunk-array).

// reliable update residual: r64 = b - Ax (when given) ; partial |r64|^2 ; r_lo = (float) r64 when given
__global__ void __launch_bounds__(256)
k_residual64(const double2* b, const double2* Ax, double2* r64, float4* r_lo, int64_t n5, double* partial,
             const int* mask) {
  __shared__ double red[16];
  const int rhs = blockIdx.y;
  if (mask && mask[rhs] == 0) return;
  b += (int64_t)rhs * 12 * n5;
  Ax += (int64_t)rhs * 12 * n5;
  if (r64) r64 += (int64_t)rhs * 12 * n5;
  if (r_lo) r_lo += (int64_t)rhs * 6 * n5;
  double loc = 0;
  for (int64_t f = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; f < 6 * n5; f += (int64_t)gridDim.x * blockDim.x) {
    const int64_t j = f / n5, i = f - j * n5;
    const int64_t ia = 2 * j * n5 + i, ib = ia + n5;
    const double2 b0 = b[ia], b1 = b[ib], a0 = Ax[ia], a1 = Ax[ib];
    const double2 o0 = make_double2(b0.x - a0.x, b0.y - a0.y), o1 = make_double2(b1.x - a1.x, b1.y - a1.y);
    if (r64) {
      r64[ia] = o0;
      r64[ib] = o1;
    }
    loc += o0.x * o0.x + o0.y * o0.y + o1.x * o1.x + o1.y * o1.y;
    if (r_lo) r_lo[f] = make_float4((float)o0.x, (float)o0.y, (float)o1.x, (float)o1.y);
  }
  const double tot = block_sum(loc, red);
  if (threadIdx.x == 0) partial[(int64_t)rhs * gridDim.x + blockIdx.x] = tot;
}

// x64 += x_lo ; x_lo = 0
__global__ void k_accum_lo(double2* x64, float4* xlo, int64_t n5, const int* mask) {
  const int rhs = blockIdx.y;
  if (mask && mask[rhs] == 0) return;
  x64 += (int64_t)rhs * 12 * n5;
  xlo += (int64_t)rhs * 6 * n5;
  for (int64_t f = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; f < 6 * n5; f += (int64_t)gridDim.x * blockDim.x) {
    const int64_t j = f / n5, i = f - j * n5;
    const int64_t ia = 2 * j * n5 + i, ib = ia + n5;
    const float4 v = xlo[f];
    double2 a = x64[ia], c = x64[ib];
    a.x += v.x; a.y += v.y; c.x += v.z; c.y += v.w;
    x64[ia] = a;
    x64[ib] = c;
    xlo[f] = make_float4(0.f, 0.f, 0.f, 0.f);
  }
}

// FP64 field -> FP32 field
__global__ void k_f64_to_f32(const double2* a, float4* o, int64_t n5, const int* mask) {
  const int rhs = blockIdx.y;
  if (mask && mask[rhs] == 0) return;
  a += (int64_t)rhs * 12 * n5;
  o += (int64_t)rhs * 6 * n5;
  for (int64_t f = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; f < 6 * n5; f += (int64_t)gridDim.x * blockDim.x) {
    const int64_t j = f / n5, i = f - j * n5;
    const double2 u = a[2 * j * n5 + i], v = a[(2 * j + 1) * n5 + i];
    o[f] = make_float4((float)u.x, (float)u.y, (float)v.x, (float)v.y);
  }
}

void cg_update(hipStream_t st, Prec p, void* x, const void* pv, const void* r, const void* q, void* rn, int64_t nreal,
               const double* scal, int alpha_slot, double* partial, int64_t nblocks, const Batch& bt) {
  const dim3 grid((unsigned)nblocks, (unsigned)bt.n);
  if (p == Prec::F32)
    hipLaunchKernelGGL(k_cg_update<float4>, grid, dim3(256), 0, st, (float4*)x, (const float4*)pv, (const float4*)r,
                       (const float4*)q, (float4*)rn, nreal / 4, scal, alpha_slot, partial, bt.mask);
  else
    hipLaunchKernelGGL(k_cg_update<double2>, grid, dim3(256), 0, st, (double2*)x, (const double2*)pv,
                       (const double2*)r, (const double2*)q, (double2*)rn, nreal / 2, scal, alpha_slot, partial,
                       bt.mask);
  LAUNCH_CHECK();
}

void dot2(hipStream_t st, Prec p, const void* a, const void* b1, const void* b2, int64_t nreal, double* partial1,
          double* partial2, int64_t nblocks, const Batch& bt) {
  const dim3 grid((unsigned)nblocks, (unsigned)bt.n);
  if (p == Prec::F32)
    hipLaunchKernelGGL(k_dot2<float4>, grid, dim3(256), 0, st, (const float4*)a, (const float4*)b1,
                       (const float4*)b2, nreal / 4, partial1, partial2, bt.mask);
  else
    hipLaunchKernelGGL(k_dot2<double2>, grid, dim3(256), 0, st, (const double2*)a, (const double2*)b1,
                       (const double2*)b2, nreal / 2, partial1, partial2, bt.mask);
  LAUNCH_CHECK();
}

void residual64(hipStream_t st, const double* b, const double* Ax, double* r64, float* r_lo, int64_t n5,
                double* partial, int64_t nblocks, const Batch& bt) {
  hipLaunchKernelGGL(k_residual64, dim3((unsigned)nblocks, (unsigned)bt.n), dim3(256), 0, st, (const double2*)b,
                     (const double2*)Ax, (double2*)r64, (float4*)r_lo, n5, partial, bt.mask);
  LAUNCH_CHECK();
}

void accum_lo(hipStream_t st, double* x64, float* xlo, int64_t n5, const Batch& bt) {
  hipLaunchKernelGGL(k_accum_lo, dim3(2048, (unsigned)bt.n), dim3(256), 0, st, (double2*)x64, (float4*)xlo, n5,
                     bt.mask);
  LAUNCH_CHECK();
}

void f64_to_f32(hipStream_t st, const double* a, float* b, int64_t n5, const Batch& bt) {
  hipLaunchKernelGGL(k_f64_to_f32, dim3(2048, (unsigned)bt.n), dim3(256), 0, st, (const double2*)a, (float4*)b, n5,
                     bt.mask);
  LAUNCH_CHECK();
}

// ---------------------------------------------------------------- scalars
//
// k_finish reduces one or two partial arrays in a fixed order and updates the
// solver scalars in `scal` (slots in kernels.h); one workgroup per RHS:
//   FIN_STORE : scal[slot] = S1
//   FIN_ALPHA : scal[PAP] = S1, alpha = rho / pAp
//   FIN_RHO   : scal[RHO] = S1
//   FIN_BETA_FR: rz = S1, beta = rz / rho, rho = rz
//   FIN_BETA_PR: rz = S1, rzold = S2, beta = (rz - rzold) / rho, rho = rz
// With p1 null, S1 = scal[slot].
__global__ void k_finish(const double* p1, const double* p2, int64_t n, double* scal, int mode, int slot,
                         const int* mask) {
  __shared__ double red[16];
  const int rhs = blockIdx.x;
  if (mask && mask[rhs] == 0) return;
  scal += (int64_t)rhs * SLOT_COUNT;
  if (p1) p1 += (int64_t)rhs * n;
  if (p2) p2 += (int64_t)rhs * n;
  double v1 = 0, v2 = 0;
  if (p1)
    for (int64_t i = threadIdx.x; i < n; i += blockDim.x) {
      v1 += p1[i];
      if (p2) v2 += p2[i];
    }
  const double r1 = block_sum(v1, red);
  const double s1 = p1 ? r1 : scal[slot];
  const double s2 = p2 ? block_sum(v2, red) : 0.0;
  if (threadIdx.x != 0) return;
  switch (mode) {
    case FIN_STORE: scal[slot] = s1; break;
    case FIN_ALPHA: scal[SLOT_PAP] = s1; scal[SLOT_ALPHA] = scal[SLOT_RHO] / s1; break;
    case FIN_RHO: scal[SLOT_RHO] = s1; break;
    case FIN_BETA_FR:
      scal[SLOT_RZ] = s1;
      scal[SLOT_BETA] = s1 / scal[SLOT_RHO];
      scal[SLOT_RHO] = s1;
      break;
    case FIN_BETA_PR:
      scal[SLOT_RZ] = s1;
      scal[SLOT_RZOLD] = s2;
      scal[SLOT_BETA] = (s1 - s2) / scal[SLOT_RHO];
      scal[SLOT_RHO] = s1;
      break;
  }
}

void finish(hipStream_t st, const double* p1, const double* p2, int64_t n, double* scal, int mode, int slot,
            const Batch& bt) {
  hipLaunchKernelGGL(k_finish, dim3((unsigned)bt.n), dim3(1024), 0, st, p1, p2, n, scal, mode, slot, bt.mask);
  LAUNCH_CHECK();
}

// ---------------------------------------------------------------- per-RHS control
//
// One thread per RHS.  The decisions are those of the outer PCG with
// reliable updates (Sec. 3.2): the iterated residual triggers a reliable
// update when it falls below delta times the largest residual since the last
// one, on convergence, or at the iteration limit; convergence is decided on
// the true residual that the update recomputes.

__global__ void k_ctl_init(Ctl c, double* scal, int n, int* join) {
  const int r = blockIdx.x * blockDim.x + threadIdx.x;
  if (r >= n || (join && !join[r])) return;
  double* sc = scal + (int64_t)r * SLOT_COUNT;
  const double bn2 = sc[SLOT_TMP];
  c.iters[r] = 0;
  c.rus[r] = 0;
  c.precs[r] = 0;
  c.ru[r] = 0;
  c.bzero[r] = 0;
  c.bnorm[r] = 0;
  c.rmax[r] = 0;
  c.rr[r] = 0;
  if (!isfinite(bn2)) {
    c.status[r] = RHS_BREAKDOWN;
    c.active[r] = 0;
  } else if (bn2 == 0.0) {
    c.status[r] = RHS_OK;
    c.active[r] = 0;
    c.bzero[r] = 1;
  } else {
    c.status[r] = RHS_RUNNING;
    c.active[r] = 1;
    c.bnorm[r] = sqrt(bn2);
  }
  sc[SLOT_TMP] = 0.0;   // beta of the first search direction p = z + 0 p
  if (join) join[r] = c.active[r];   // the start-up kernels that follow run on these RHS only
}

__global__ void k_ctl_start(Ctl c, const double* scal, int n, int has_x0, const int* join) {
  const int r = blockIdx.x * blockDim.x + threadIdx.x;
  if (r >= n || !c.active[r] || (join && !join[r])) return;
  const double bn = c.bnorm[r];
  const double rr = has_x0 ? scal[(int64_t)r * SLOT_COUNT + SLOT_R64] : bn * bn;
  c.rr[r] = has_x0 ? rr : bn * bn;
  c.rmax[r] = has_x0 ? sqrt(rr) : bn;
  c.precs[r] = 1;   // the preconditioner application before the first iteration
}

__global__ void k_ctl_iterate(Ctl c, const double* scal, int n, CtlParams p) {
  const int r = blockIdx.x * blockDim.x + threadIdx.x;
  if (r >= n || !c.active[r]) return;
  const double* sc = scal + (int64_t)r * SLOT_COUNT;
  const double pap = sc[SLOT_PAP], rr = sc[SLOT_RR];
  c.iters[r] += 1;
  c.rr[r] = rr;
  if (!(pap > 0.0) || !isfinite(pap) || !isfinite(rr)) {
    c.status[r] = RHS_BREAKDOWN;
    c.active[r] = 0;
    c.ru[r] = 0;
    return;
  }
  const double rn = sqrt(rr);
  if (rn > c.rmax[r]) c.rmax[r] = rn;
  const bool conv = rn <= p.tol * c.bnorm[r];
  const bool last = c.iters[r] >= p.maxiter;
  c.ru[r] = (conv || last || (p.delta > 0 && rn < p.delta * c.rmax[r])) ? 1 : 0;
}

__global__ void __launch_bounds__(1024) k_ctl_after_update(Ctl c, double* scal, int n, CtlParams p) {
  __shared__ int cnt;
  if (threadIdx.x == 0) cnt = 0;
  __syncthreads();
  for (int r = threadIdx.x; r < n; r += blockDim.x) {
    if (!c.active[r]) continue;
    double* sc = scal + (int64_t)r * SLOT_COUNT;
    if (c.ru[r]) {
      const double rr = sc[SLOT_R64];
      c.ru[r] = 0;
      c.rus[r] += 1;
      c.rr[r] = rr;
      sc[SLOT_RR] = rr;   // the current |r|^2 is the true one
      c.rmax[r] = sqrt(rr);
      if (sqrt(rr) <= p.tol * c.bnorm[r]) {
        c.status[r] = RHS_OK;
        c.active[r] = 0;
        continue;
      }
      if (!isfinite(rr)) {
        c.status[r] = RHS_BREAKDOWN;
        c.active[r] = 0;
        continue;
      }
    }
    if (c.iters[r] >= p.maxiter) {
      c.status[r] = RHS_NOT_CONVERGED;
      c.active[r] = 0;
      continue;
    }
    c.precs[r] += 1;
    atomicAdd(&cnt, 1);
  }
  __syncthreads();
  if (threadIdx.x == 0) *c.nactive = cnt;
}

static unsigned ctl_blocks(int n) { return (unsigned)((n + 255) / 256); }

void ctl_init(hipStream_t st, const Ctl& c, double* scal, int n, int* join) {
  hipLaunchKernelGGL(k_ctl_init, dim3(ctl_blocks(n)), dim3(256), 0, st, c, scal, n, join);
  LAUNCH_CHECK();
}

void ctl_start(hipStream_t st, const Ctl& c, const double* scal, int n, bool has_x0, const int* join) {
  hipLaunchKernelGGL(k_ctl_start, dim3(ctl_blocks(n)), dim3(256), 0, st, c, scal, n, has_x0 ? 1 : 0, join);
  LAUNCH_CHECK();
}

void ctl_iterate(hipStream_t st, const Ctl& c, const double* scal, int n, const CtlParams& p) {
  hipLaunchKernelGGL(k_ctl_iterate, dim3(ctl_blocks(n)), dim3(256), 0, st, c, scal, n, p);
  LAUNCH_CHECK();
}

void ctl_after_update(hipStream_t st, const Ctl& c, double* scal, int n, const CtlParams& p) {
  hipLaunchKernelGGL(k_ctl_after_update, dim3(1), dim3(1024), 0, st, c, scal, n, p);
  LAUNCH_CHECK();
}

}  // namespace mspcg
