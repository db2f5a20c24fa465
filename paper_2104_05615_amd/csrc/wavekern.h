// One hop with the fused fifth-dimension epilogue, a wavefront per 16 output
// sites, or (at the end) a lane per 5D output site.  The general kernel is
// k_hop in sitekern.h; results are the same bit for bit.
//
// For Ls = 4 LC <= 16 a wavefront owns 16 sites x Ls slices by itself: lane
// 4 j + g works on the slices s = 4 r + g, r < LC, of site j.  The four lanes
// of a site read 64 consecutive bytes per load, a term's link is loaded once
// for the LC slices of a lane, and the workgroup is that one wavefront, so
// nothing waits at a barrier for the slowest of several wavefronts.
#pragma once

#include "sitekern.h"

namespace mspcg {

// f(integral_constant<0>) ... f(integral_constant<N - 1>)
template <typename F, int... I> __device__ __forceinline__ void static_for_seq(F&& f, std::integer_sequence<int, I...>) {
  (f(std::integral_constant<int, I>()), ...);
}
template <int N, typename F> __device__ __forceinline__ void static_for(F&& f) {
  static_for_seq(f, std::make_integer_sequence<int, N>());
}

// Bit set in the byte offsets of an absent term's loads: past the end of every
// chunk array (below 4 GiB / 3 per chunk), scale array (offset / 4 or / 2) and
// FP32 or FP16 link array (below 2^31 bytes), and no sum with an offset inside
// wraps, so the reads return zeros and stores are dropped.
constexpr uint32_t kAbsent = 0x80000000u;

// Staging tile of a wavefront in LDS: 16 sites of Ls rows of 48 bytes (24
// 16-bit or 12 32-bit components).  The padding of a site spreads the 16-byte
// accesses of the 8 lanes served together over distinct banks, both in the
// hop's lane order (site lane / 4) and in the MFMA's (site lane % 16).
template <int LC> constexpr int wave_tile_stride() { return LC * 192 + (LC == 1 ? 32 : LC == 2 ? 48 : 16); }

// ---------------------------------------------------------------- neighbours

// A wavefront's view of a geometry: where term k (2 mu: forward, 2 mu + 1:
// backward) of the lane's site reads its spinor and its link.
template <typename Geo> struct WaveSite;

template <typename T, typename L, bool M> struct WaveSite<SubGeo<T, L, M>> {
  using Geo = SubGeo<T, L, M>;
  int nb[8], gco[4];
  uint32_t lx, base_in;
  __device__ __forceinline__ WaveSite(const Geo& g, const SiteRef& r) {
    const uint32_t site = r.valid ? (uint32_t)r.site : 0u;
    const short4 o = g.tb.origin[r.d];
    const short4 lc = g.tb.coords[site];
    const int4 n0 = reinterpret_cast<const int4*>(g.tb.nbr)[2 * site];
    const int4 n1 = reinterpret_cast<const int4*>(g.tb.nbr)[2 * site + 1];
    const int n[8] = {n0.x, n0.y, n0.z, n0.w, n1.x, n1.y, n1.z, n1.w};
#pragma unroll
    for (int k = 0; k < 8; ++k) nb[k] = r.valid ? n[k] : -1;
    const int l[4] = {o.x + lc.x, o.y + lc.y, o.z + lc.z, o.w + lc.w};
#pragma unroll
    for (int m = 0; m < 4; ++m) {
      int v = l[m];
      if (v < 0) v += g.tb.dims[m];
      if (v >= g.tb.dims[m]) v -= g.tb.dims[m];
      gco[m] = v;
    }
    lx = g.lat.lex(gco);
    base_in = (uint32_t)r.d * (uint32_t)g.tb.n_in;
  }
  // terms that at least one site of the wavefront has
  __device__ __forceinline__ uint32_t mask() const {
    uint32_t m = 0;
#pragma unroll
    for (int k = 0; k < 8; ++k) m |= __builtin_amdgcn_ballot_w64(nb[k] >= 0) != 0 ? 1u << k : 0u;
    return m;
  }
  template <int K> __device__ __forceinline__ uint32_t absent() const { return (uint32_t)nb[K] & kAbsent; }
  template <int K> __device__ __forceinline__ uint32_t in_site(const Geo& g) const {
    return base_in + (uint32_t)max(nb[K], 0);
  }
  template <int K> __device__ __forceinline__ uint32_t link_site(const Geo& g) const {
    constexpr int MU = K / 2;
    if constexpr (K % 2 == 0) return lx >> 1;
    const uint32_t st = g.lat.stride(MU);
    return (lx + (gco[MU] == 0 ? (uint32_t)(g.lat.ext(MU) - 1) * st : 0u - st)) >> 1;
  }
};

// ---------------------------------------------------------------- loads

// one buffer resource per chunk array: a site's chunks are then read at one
// vector offset plus immediates
template <typename S> struct ChunkRsrc {
  static constexpr int N = StoreTraits<S>::nchunk;
  __amdgpu_buffer_rsrc_t c[N], sc;
  __device__ __forceinline__ ChunkRsrc(const Field<S>& f) {
    using C = typename Field<S>::chunk;
#pragma unroll
    for (int k = 0; k < N; ++k) c[k] = make_rsrc(f.data + (int64_t)k * f.stride, (uint64_t)f.stride * sizeof(C));
    if constexpr (StoreTraits<S>::scaled) sc = make_rsrc(f.scale, (uint64_t)f.stride * 4u);
  }
};

// a lane's stored components of one 5D site
template <typename S> struct Raw;
template <> struct Raw<float> {
  u32x4 q[6];
  __device__ __forceinline__ void load(const ChunkRsrc<float>& f, uint32_t off) {
#pragma unroll
    for (int k = 0; k < 6; ++k) q[k] = __builtin_amdgcn_raw_buffer_load_b128(f.c[k], off, 0, 0);
  }
  __device__ __forceinline__ void values(float* v) const {
#pragma unroll
    for (int k = 0; k < 6; ++k) {
      v[4 * k] = __uint_as_float(q[k].x);
      v[4 * k + 1] = __uint_as_float(q[k].y);
      v[4 * k + 2] = __uint_as_float(q[k].z);
      v[4 * k + 3] = __uint_as_float(q[k].w);
    }
  }
};
template <> struct Raw<__half> {
  u32x4 q[3];
  float s;
  __device__ __forceinline__ void load(const ChunkRsrc<__half>& f, uint32_t off) {
#pragma unroll
    for (int k = 0; k < 3; ++k) q[k] = __builtin_amdgcn_raw_buffer_load_b128(f.c[k], off, 0, 0);
    s = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(f.sc, off >> 2, 0, 0));
  }
  __device__ __forceinline__ u32x4 halves(int k) const { return q[k]; }
  __device__ __forceinline__ void values(float* v) const {
#pragma unroll
    for (int k = 0; k < 12; ++k) {
      const uint32_t w = q[k >> 2][k & 3];
      v[2 * k] = half_lo(w) * s;
      v[2 * k + 1] = half_hi(w) * s;
    }
  }
};
template <> struct Raw<int8_t> {
  u32x2 q[3];
  float s;
  __device__ __forceinline__ void load(const ChunkRsrc<int8_t>& f, uint32_t off) {
#pragma unroll
    for (int k = 0; k < 3; ++k) q[k] = __builtin_amdgcn_raw_buffer_load_b64(f.c[k], off, 0, 0);
    s = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(f.sc, off >> 1, 0, 0));
  }
  __device__ __forceinline__ u32x4 halves(int k) const { return i8_to_h16(q[k]); }
  __device__ __forceinline__ void values(float* v) const {
    float t[24];
#pragma unroll
    for (int k = 0; k < 3; ++k) unpack8_i8(make_uint2(q[k].x, q[k].y), t + 8 * k);
#pragma unroll
    for (int k = 0; k < 24; ++k) v[k] = t[k] * s;
  }
};

// No instruction is scheduled across this point (left to itself, the compiler
// issues all loads of a hop at once and spills, or each shortly before its use).
__device__ __forceinline__ void sched_fence() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_sched_barrier(0);
}
// ... and these accumulators are final here
__device__ __forceinline__ void pin24(float* a) {
#pragma unroll
  for (int k = 0; k < 24; ++k) asm volatile("" : "+v"(a[k]));
  sched_fence();
}

// ---------------------------------------------------------------- hop

// acc[r] = the hop at slice 4 r + g of the lane's site.  Terms in the order
// of the general kernel; an absent term's loads return zeros.
template <int LC, bool DAG, typename Geo, typename S>
__device__ __forceinline__ void wave_hop(const Geo& geo, const WaveSite<Geo>& ws, const Field<S>& in, int g,
                                         float (&acc)[LC][24]) {
  constexpr uint32_t CB = sizeof(typename Field<S>::chunk);
  const ChunkRsrc<S> rs(in);
  const uint32_t mask = ws.mask();
#pragma unroll
  for (int r = 0; r < LC; ++r)
#pragma unroll
    for (int k = 0; k < 24; ++k) acc[r][k] = 0.f;
  auto spinor_off = [&](auto kc) -> uint32_t {
    constexpr int K = decltype(kc)::value;
    return ((ws.template in_site<K>(geo) * (4u * LC) + (uint32_t)g) * CB) | ws.template absent<K>();
  };
  auto link_off = [&](auto kc, uint32_t rec) -> uint32_t {
    constexpr int K = decltype(kc)::value;
    const uint32_t par = K % 2 == 0 ? geo.par : 1 - geo.par;
    return (((par * 4 + K / 2) * (uint32_t)geo.g.vh + ws.template link_site<K>(geo)) * rec) | ws.template absent<K>();
  };
  if constexpr (std::is_same<S, float>::value) {
    // FP32: steps (term, r), the spinors of the next DEPTH steps and the next
    // term's link in flight
    const __amdgpu_buffer_rsrc_t lr = make_rsrc(geo.g.data, (uint64_t)80 * (uint64_t)geo.g.vh * 8u);
    constexpr int DEPTH = LC == 2 || LC == 3 ? 3 : 2, NS = 8 * LC;
    Raw<float> q[DEPTH];
    u32x4 lw[2][5];
    uint32_t soff[2];
    auto issue = [&](auto sc) {
      constexpr int st = decltype(sc)::value;
      if constexpr (st < NS) {
        constexpr int K = st / LC, R = st % LC;
        const auto kc = std::integral_constant<int, K>();
        if (mask >> K & 1) {
          if constexpr (R == 0) {
            soff[K & 1] = spinor_off(kc);
            const uint32_t lo = link_off(kc, 80u);
#pragma unroll
            for (int i = 0; i < 5; ++i) lw[K & 1][i] = __builtin_amdgcn_raw_buffer_load_b128(lr, lo + 16 * i, 0, 0);
          }
          q[st % DEPTH].load(rs, soff[K & 1] + R * 4 * CB);
        }
        sched_fence();
      }
    };
    static_for<DEPTH - 1>([&](auto sc) { issue(sc); });
    static_for<NS>([&](auto sc) {
      constexpr int st = decltype(sc)::value, K = st / LC, R = st % LC;
      issue(std::integral_constant<int, st + DEPTH - 1>());
      if (mask >> K & 1) {
        constexpr bool FWD = K % 2 == 0;
        constexpr int SIGN = (FWD ? -1 : 1) * (DAG ? -1 : 1);
        float psi[24], h[12], gh[12], u[18];
        q[st % DEPTH].values(psi);
#pragma unroll
        for (int i = 0; i < 18; ++i) u[i] = __uint_as_float(lw[K & 1][i >> 2][i & 3]);
        project<K / 2, SIGN>(psi, h);
        su3_mul_half<!FWD>(u, h, gh);
        reconstruct_add<K / 2, SIGN>(gh, acc[R]);
      }
      pin24(acc[R]);
    });
  } else {
    // 16- and 8-bit formats: the SU(3) products run on v_mfma_f32_4x4x4f16,
    // a block's four lanes being the four lanes of one site; the next term's
    // spinors and link words are in flight
    const __amdgpu_buffer_rsrc_t lr = make_rsrc(geo.g.data, (uint64_t)80 * (uint64_t)geo.g.vh * 4u);
    const uint32_t a = (uint32_t)min(g, 2);
    Raw<S> q[2][LC];
    u32x4 lw[2];
    auto issue = [&](auto kc) {
      constexpr int K = decltype(kc)::value;
      if constexpr (K < 8) {
        if (mask >> K & 1) {
          const uint32_t lo = link_off(kc, 40u) + 4u * (K % 2 == 0 ? 3 * a : a);
          constexpr uint32_t step = K % 2 == 0 ? 4 : 12;
          lw[K & 1].x = __builtin_amdgcn_raw_buffer_load_b32(lr, lo, 0, 0);
          lw[K & 1].y = __builtin_amdgcn_raw_buffer_load_b32(lr, lo + step, 0, 0);
          lw[K & 1].z = __builtin_amdgcn_raw_buffer_load_b32(lr, lo + 2 * step, 0, 0);
          const uint32_t so = spinor_off(kc);
#pragma unroll
          for (int r = 0; r < LC; ++r) q[K & 1][r].load(rs, so + r * 4 * CB);
        }
        sched_fence();
      }
    };
    issue(std::integral_constant<int, 0>());
    static_for<8>([&](auto kc) {
      constexpr int K = decltype(kc)::value;
      issue(std::integral_constant<int, K + 1>());
      if (mask >> K & 1) {
        constexpr bool FWD = K % 2 == 0;
        constexpr int SIGN = (FWD ? -1 : 1) * (DAG ? -1 : 1);
#pragma unroll
        for (int r = 0; r < LC; ++r) {
          const Raw<S>& p = q[K & 1][r];
          term_mfma<K / 2, SIGN, !FWD>(p.halves(0), p.halves(1), p.halves(2), lw[K & 1], p.s, acc[r]);
        }
      }
#pragma unroll
      for (int r = 0; r < LC; ++r) pin24(acc[r]);
    });
  }
}

// ---------------------------------------------------------------- epilogue

// The sum of the 16 Ls values of buf (LDS, index site * Ls + s) in the order of
// the general kernel, whose threads are (site, s), s fastest: a butterfly over
// each of its LC wavefronts, then the wavefronts in turn.
template <int LC> __device__ __forceinline__ double wave_dot(const float* buf, int lane) {
  __syncthreads();
  double tot = 0;
#pragma unroll
  for (int i = 0; i < LC; ++i) {
    double v = (double)buf[64 * i + lane];
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off);
    tot += v;
  }
  return tot;
}

// 24 FP32 values as the stored form of S (three chunk words) and its scale:
// the arithmetic of store_site
template <typename S> struct Packed;
template <> struct Packed<__half> {
  using word = u32x4;
  u32x4 q[3];
  float s;
  __device__ __forceinline__ void from(const float* v) {
    float mx = 0.f;
#pragma unroll
    for (int k = 0; k < 24; ++k) mx = fmaxf(mx, fabsf(v[k]));
    const float inv = mx > 0.f ? 1.0f / mx : 0.f;
#pragma unroll
    for (int k = 0; k < 12; ++k)
      q[k >> 2][k & 3] = f2h_bits(v[2 * k] * inv) | (f2h_bits(v[2 * k + 1] * inv) << 16);
    s = mx;
  }
};
template <> struct Packed<int8_t> {
  using word = u32x2;
  u32x2 q[3];
  float s;
  __device__ __forceinline__ void from(const float* v) {
    float mx = 0.f;
#pragma unroll
    for (int k = 0; k < 24; ++k) mx = fmaxf(mx, fabsf(v[k]));
    const float inv = mx > 0.f ? 127.0f / mx : 0.f;
    float t[24];
#pragma unroll
    for (int k = 0; k < 24; ++k) t[k] = v[k] * inv;
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      const uint2 c = pack8_i8(t + 8 * k);
      q[k].x = c.x;
      q[k].y = c.y;
    }
    s = mx * (1.0f / 127.0f);
  }
};

// two products rounded to FP32 and then to a pair of halves (one packed
// conversion), as the general kernel's operands are
__device__ __forceinline__ uint32_t h2_bits(float a, float b) {
  asm("" : "+v"(a), "+v"(b));   // the product stays an FP32 number: no mixed-precision multiply to FP16
  const float2_t v = {a, b};
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, half2_t));
}

// B operands of 4 consecutive components from the FP16 tile: rows 4 g2 + v
__device__ __forceinline__ void tile_b16(const unsigned char* row0, int q0, half4_t* b) {
  u32x2 x[4];
#pragma unroll
  for (int v = 0; v < 4; ++v) x[v] = *reinterpret_cast<const u32x2*>(row0 + v * 48 + q0 * 2);
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int w = j >> 1;
    const uint32_t sel = (j & 1) ? 0x07060302u : 0x05040100u;   // the high (low) halves of two words
    b[j] = hpair(__builtin_amdgcn_perm(x[1][w], x[0][w], sel), __builtin_amdgcn_perm(x[3][w], x[2][w], sel));
  }
}

// y = E0 w (centre field, where it exists) + E1 h, h the hop, and optionally
// <dotf, y> per 16 sites (8-bit format only: FP32 and FP16 have no adjoint hop
// here); E1 is never null, E0 with HASW neither.
//
// What bounds it: a region hop's reads through the L1 (every spinor is read
// by up to eight sites) and, at the rim sites with one or two of the eight
// terms, the epilogue.  The term loop skips what no site of the wavefront has by
// a scalar branch (the regions are ordered by neighbour pattern), and nothing
// but the wavefront itself waits in the epilogue: h2 (N2 <- N1, 12 FP16 slices,
// 256 subdomains of 8^3x16) 1867 -> 1542 us, at 256 of 4^3x8 211 -> 160 us.
template <typename Geo, typename S, int LC, bool DAG, bool HASW>
__global__ void __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(2)))
k_hop_wave(Geo geo, Field<S> out_b, Field<S> in_b, Field<S> w_b, Field<S> dotf_b, const float* E0, const float* E1,
           double* dot_partial, HopWork wk) {
  constexpr int Ls = 4 * LC, STR = wave_tile_stride<LC>();
  constexpr uint32_t CB = sizeof(typename Field<S>::chunk);
  __shared__ __align__(16) unsigned char tile[16 * STR];
  const int lane = threadIdx.x;
  const int j = lane >> 2, g = lane & 3;        // hop: site, slices 4 r + g
  const int col = lane & 15, g2 = lane >> 4;    // MFMA: site column, row group
  int64_t blk;
  int rhs;
  wk.decode(blockIdx.x, gridDim.x, blk, rhs);
  if (wk.mask && wk.mask[rhs] == 0) return;   // uniform over the workgroup
  blk = geo.physical(blk);
  const Field<S> out = out_b.at(rhs), in = in_b.at(rhs);
  const SiteRef ref = geo.locate(blk, j, 16, Ls, g);
  const WaveSite<Geo> ws(geo, ref);
  float acc[LC][24];
  wave_hop<LC, DAG>(geo, ws, in, g, acc);

  constexpr bool DOT = DAG && HASW;
  const ChunkRsrc<S> ro(out);
  const uint32_t oo = ref.valid ? (uint32_t)ref.out5 * CB : kAbsent;
  const uint32_t wo = HASW && ref.valid && ref.w5 >= 0 ? (uint32_t)ref.w5 * CB : kAbsent;
  unsigned char* mine = tile + j * STR + g * 48;   // + r * 192: the lane's rows

  if constexpr (std::is_same<S, float>::value) {
    // FP32: one chirality (12 components, 48-byte rows) at a time
    static_assert(!DAG, "FP32: no fused dot");
    const int ic = min(col, Ls - 1);
#pragma unroll
    for (int chi = 0; chi < 2; ++chi) {
      u32x4 wq[LC][3];
      if constexpr (HASW) {
        const ChunkRsrc<S> rw(w_b.at(rhs));
#pragma unroll
        for (int r = 0; r < LC; ++r)
#pragma unroll
          for (int k = 0; k < 3; ++k)
            wq[r][k] = __builtin_amdgcn_raw_buffer_load_b128(rw.c[3 * chi + k], wo + r * 4 * CB, 0, 0);
      }
      float4_t d[12];
#pragma unroll
      for (int k = 0; k < 12; ++k) d[k] = float4_t{0.f, 0.f, 0.f, 0.f};
      auto product = [&](const float* E) {
        float a[LC];
#pragma unroll
        for (int kk = 0; kk < LC; ++kk) {
          const float e = E[(chi * Ls + ic) * Ls + 4 * kk + g2];
          a[kk] = col < Ls ? e : 0.f;
        }
        __syncthreads();
        const unsigned char* b = tile + col * STR + g2 * 48;
#pragma unroll
        for (int q = 0; q < 3; ++q)
#pragma unroll
          for (int kk = 0; kk < LC; ++kk) {
            const float4_t x = *reinterpret_cast<const float4_t*>(b + kk * 192 + q * 16);
#pragma unroll
            for (int i = 0; i < 4; ++i)
              d[4 * q + i] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[kk], x[i], d[4 * q + i], 0, 0, 0);
          }
        __syncthreads();
      };
#pragma unroll
      for (int r = 0; r < LC; ++r)
#pragma unroll
        for (int k = 0; k < 3; ++k) {
          const float* h = acc[r] + 12 * chi + 4 * k;
          *reinterpret_cast<float4_t*>(mine + r * 192 + k * 16) = float4_t{h[0], h[1], h[2], h[3]};
        }
      product(E1);
      if constexpr (HASW) {
#pragma unroll
        for (int r = 0; r < LC; ++r)
#pragma unroll
          for (int k = 0; k < 3; ++k) *reinterpret_cast<u32x4*>(mine + r * 192 + k * 16) = wq[r][k];
        product(E0);
      }
      // rows 4 g2 + v of site column col
      if (g2 < LC) {
        unsigned char* o = tile + col * STR + g2 * 192;
#pragma unroll
        for (int v = 0; v < 4; ++v)
#pragma unroll
          for (int q = 0; q < 3; ++q)
            *reinterpret_cast<float4_t*>(o + v * 48 + q * 16) =
                float4_t{d[4 * q][v], d[4 * q + 1][v], d[4 * q + 2][v], d[4 * q + 3][v]};
      }
      __syncthreads();
#pragma unroll
      for (int r = 0; r < LC; ++r)
#pragma unroll
        for (int k = 0; k < 3; ++k) {
          const u32x4 c = *reinterpret_cast<const u32x4*>(mine + r * 192 + k * 16);
          __builtin_amdgcn_raw_buffer_store_b128(c, ro.c[3 * chi + k], oo + r * 4 * CB, 0, 0);
        }
      __syncthreads();
    }
  } else {
    // FP16 operands: every site column scaled by its largest entry; the rows
    // of the centre field are first rounded over their own largest entry
    float rowmax[LC];
    uint32_t wp[LC][12];
    bool live = false;   // some site of the wavefront has a centre field
#pragma unroll
    for (int r = 0; r < LC; ++r) rowmax[r] = 0.f;
    if constexpr (HASW) {
      live = __builtin_amdgcn_ballot_w64(wo != kAbsent) != 0;
      if (live) {
        const ChunkRsrc<S> rw(w_b.at(rhs));
        Raw<S> wq[LC];
#pragma unroll
        for (int r = 0; r < LC; ++r) wq[r].load(rw, wo + r * 4 * CB);
#pragma unroll
        for (int r = 0; r < LC; ++r) {
          float v[24];
          wq[r].values(v);
          float m = 0.f;
#pragma unroll
          for (int k = 0; k < 24; ++k) m = fmaxf(m, fabsf(v[k]));
          const float im = m > 0.f ? 1.f / m : 0.f;
#pragma unroll
          for (int k = 0; k < 12; ++k) wp[r][k] = h2_bits(v[2 * k] * im, v[2 * k + 1] * im);
          rowmax[r] = m;
        }
      }
    }
    float cs = 0.f;
#pragma unroll
    for (int r = 0; r < LC; ++r) {
#pragma unroll
      for (int k = 0; k < 24; ++k) cs = fmaxf(cs, fabsf(acc[r][k]));
      cs = fmaxf(cs, rowmax[r]);
    }
    cs = fmaxf(cs, __shfl_xor(cs, 1));
    cs = fmaxf(cs, __shfl_xor(cs, 2));
    const float ics = cs > 0.f ? 1.f / cs : 0.f;
    float4_t d[24];
#pragma unroll
    for (int k = 0; k < 24; ++k) d[k] = float4_t{0.f, 0.f, 0.f, 0.f};
    const int gc = min(g2, LC - 1), ic = min(col, Ls - 1);   // clamped: rows past Ls meet zero A entries
    const unsigned char* brow = tile + col * STR + gc * 192;
    auto product = [&](const float* E) {
      half4_t a[2];
#pragma unroll
      for (int chi = 0; chi < 2; ++chi) {
        const float4_t e = *reinterpret_cast<const float4_t*>(E + (chi * Ls + ic) * Ls + 4 * gc);
#pragma unroll
        for (int v = 0; v < 4; ++v) a[chi][v] = (col < Ls && g2 < LC) ? (_Float16)e[v] : (_Float16)0.f;
      }
      __syncthreads();
#pragma unroll
      for (int q = 0; q < 6; ++q) {
        half4_t b[4];
        tile_b16(brow, 4 * q, b);
#pragma unroll
        for (int i = 0; i < 4; ++i)
          d[4 * q + i] = __builtin_amdgcn_mfma_f32_16x16x16f16(a[q >= 3 ? 1 : 0], b[i], d[4 * q + i], 0, 0, 0);
      }
      __syncthreads();
    };
#pragma unroll
    for (int r = 0; r < LC; ++r)
#pragma unroll
      for (int k = 0; k < 3; ++k) {
        u32x4 w;
#pragma unroll
        for (int i = 0; i < 4; ++i) w[i] = h2_bits(acc[r][8 * k + 2 * i] * ics, acc[r][8 * k + 2 * i + 1] * ics);
        *reinterpret_cast<u32x4*>(mine + r * 192 + k * 16) = w;
      }
    product(E1);
    if (live) {
#pragma unroll
      for (int r = 0; r < LC; ++r) {
        const float rsw = rowmax[r] * ics;
#pragma unroll
        for (int k = 0; k < 3; ++k) {
          u32x4 w;
#pragma unroll
          for (int i = 0; i < 4; ++i)
            w[i] = h2_bits(half_lo(wp[r][4 * k + i]) * rsw, half_hi(wp[r][4 * k + i]) * rsw);
          *reinterpret_cast<u32x4*>(mine + r * 192 + k * 16) = w;
        }
      }
      product(E0);
    }
    // rows 4 g2 + v of site column col, in their stored form
    const float csc = __shfl(cs, 4 * col);
    const SiteRef oref = geo.locate(blk, col, 16, Ls, 0);   // the column's site
    const bool own = g2 < LC;
    const uint32_t oi = own && oref.valid ? (uint32_t)oref.out5 + 4u * g2 : 0u;
    const uint32_t off = own && oref.valid ? 0u : kAbsent;
    float osc[4], loc[4];
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      float y[24];
#pragma unroll
      for (int k = 0; k < 24; ++k) y[k] = d[k][v] * csc;
      Packed<S> pk;
      pk.from(y);
      osc[v] = pk.s;
      if (own) {
#pragma unroll
        for (int k = 0; k < 3; ++k)
          *reinterpret_cast<typename Packed<S>::word*>(tile + col * STR + (4 * g2 + v) * 48 + k * 16) = pk.q[k];
      }
      loc[v] = 0.f;
      if constexpr (DOT) {
        if (dot_partial) {
          const ChunkRsrc<S> rp(dotf_b.at(rhs));
          Raw<S> pq;
          pq.load(rp, (oi + v) * CB | off);
          float pv[24];
          pq.values(pv);
#pragma unroll
          for (int k = 0; k < 24; ++k) loc[v] += pv[k] * y[k];
        }
      }
    }
    u32x4 sw;
#pragma unroll
    for (int v = 0; v < 4; ++v) sw[v] = __float_as_uint(osc[v]);
    __builtin_amdgcn_raw_buffer_store_b128(sw, ro.sc, oi * 4u | off, 0, 0);
    __syncthreads();
#pragma unroll
    for (int r = 0; r < LC; ++r)
#pragma unroll
      for (int k = 0; k < 3; ++k) {
        const auto c = *reinterpret_cast<const typename Packed<S>::word*>(mine + r * 192 + k * 16);
        if constexpr (std::is_same<S, __half>::value)
          __builtin_amdgcn_raw_buffer_store_b128(c, ro.c[k], oo + r * 4 * CB, 0, 0);
        else
          __builtin_amdgcn_raw_buffer_store_b64(c, ro.c[k], oo + r * 4 * CB, 0, 0);
      }
    if constexpr (DOT) {
      if (dot_partial) {
        float* buf = reinterpret_cast<float*>(tile);
        __syncthreads();
        if (own) {
#pragma unroll
          for (int v = 0; v < 4; ++v) buf[col * Ls + 4 * g2 + v] = oref.valid ? loc[v] : 0.f;
        }
        const double tot = wave_dot<LC>(buf, lane);
        if (lane == 0) dot_partial[(int64_t)rhs * wk.nblk + blk] = tot;
      }
    }
  }
}

// ---------------------------------------------------------------- small launches

// The same hop with a wavefront per 64 / Ls sites, a lane per 5D site, for the
// 16- and 8-bit formats and Ls = 4, 8 or 16.  A workgroup has the wavefronts of
// 16 sites; they meet only in the sum of the dot.
//
// What bounds it: the length of one wavefront's instruction and memory chain,
// in launches that give each SIMD about one wavefront.  So all loads of the hop
// are in flight at once (a lane has one slice, hence registers for eight
// terms), with those of the centre field, the dot and the matrices behind them;
// and the epilogue's MFMAs have 4 sites x 4 components as rows and slices as
// columns, one group of 4 sites after the other (each in its part of the k
// range), so a lane ends with the 24 components of the 5D site that it began
// with and stores them from its registers.  Tried before it at 8^4 x 8, FP16, 16
// subdomains of 4^4: an instance of the wavefront kernel for h4, which spent
// 2000 of its 21000 cycles on the tables, 7000 on the hop, 2000 waiting for the
// centre field, 3100 on the products and 7000 on packing and the dot.  Per
// launch from the faster of the other two kernels h1 9.6 -> 8.7, h2 12.1 -> 9.9, h3
// 9.8 -> 8.8, h4 13.0 -> 8.9 us, a mixed-precision solve 31.9 -> 27.9 ms.
// LDS bytes per site; the padding spreads a wavefront's accesses over the banks
template <int Ls> constexpr int lane_site_stride() { return 24 * Ls * 2 + Ls * 2; }

template <typename Geo, typename S, int Ls, bool DAG, bool HASW>
__global__ void __launch_bounds__(16 * Ls) __attribute__((amdgpu_waves_per_eu(2)))
k_hop_lane(Geo geo, Field<S> out_b, Field<S> in_b, Field<S> w_b, Field<S> dotf_b, const float* E0, const float* E1,
           double* dot_partial, HopWork wk) {
  constexpr uint32_t CB = sizeof(typename Field<S>::chunk);
  constexpr int NS = 64 / Ls, NG = NS / 4, NW = Ls / 4, STR = lane_site_stride<Ls>();
  constexpr bool DOT = DAG && HASW;
  __shared__ __align__(16) unsigned char tiles[NW * NS * STR];
  __shared__ double red[NW];
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int col = lane & 15, g2 = lane >> 4;
  const int j = g2 + 4 * (col / Ls), s = col % Ls;   // the lane's site of the wavefront, and slice
  int64_t blk;
  int rhs;
  wk.decode(blockIdx.x, gridDim.x, blk, rhs);
  if (wk.mask && wk.mask[rhs] == 0) return;   // uniform over the workgroup
  blk = geo.physical(blk);
  const Field<S> out = out_b.at(rhs), in = in_b.at(rhs);
  const SiteRef ref = geo.locate(blk, wave * NS + j, 16, Ls, s);
  const WaveSite<Geo> ws(geo, ref);
  const uint32_t mask = ws.mask();
  const uint32_t oo = ref.valid ? (uint32_t)ref.out5 * CB : kAbsent;
  const uint32_t wo = HASW && ref.valid && ref.w5 >= 0 ? (uint32_t)ref.w5 * CB : kAbsent;
  const bool live = HASW && __builtin_amdgcn_ballot_w64(wo != kAbsent) != 0;

  const ChunkRsrc<S> rs(in);
  const __amdgpu_buffer_rsrc_t lr = make_rsrc(geo.g.data, (uint64_t)80 * (uint64_t)geo.g.vh * 4u);
  Raw<S> q[8], wq, pq;
  u32x4 lw[8];
  auto load_term = [&](auto kc) {
    constexpr int K = decltype(kc)::value;
    const uint32_t a = (uint32_t)min(lane & 3, 2), par = K % 2 == 0 ? geo.par : 1 - geo.par;
    const uint32_t lo = ((((par * 4 + K / 2) * (uint32_t)geo.g.vh + ws.template link_site<K>(geo)) * 40u) |
                         ws.template absent<K>()) + 4u * (K % 2 == 0 ? 3 * a : a);
    constexpr uint32_t step = K % 2 == 0 ? 4 : 12;
    lw[K].x = __builtin_amdgcn_raw_buffer_load_b32(lr, lo, 0, 0);
    lw[K].y = __builtin_amdgcn_raw_buffer_load_b32(lr, lo + step, 0, 0);
    lw[K].z = __builtin_amdgcn_raw_buffer_load_b32(lr, lo + 2 * step, 0, 0);
    q[K].load(rs, ((ws.template in_site<K>(geo) * (uint32_t)Ls + (uint32_t)s) * CB) | ws.template absent<K>());
  };
  // MFMA B operands: column s of the matrices, the 4 rows of this lane's k group
  const int kg = g2 % NW;
  float4_t m1[2], m0[2];
  auto load_rest = [&]() {
    if constexpr (HASW) wq.load(ChunkRsrc<S>(w_b.at(rhs)), wo);
    if constexpr (DOT) {
      if (dot_partial) pq.load(ChunkRsrc<S>(dotf_b.at(rhs)), oo);
    }
#pragma unroll
    for (int chi = 0; chi < 2; ++chi) {
      m1[chi] = *reinterpret_cast<const float4_t*>(E1 + (chi * Ls + s) * Ls + 4 * kg);
      if constexpr (HASW) m0[chi] = *reinterpret_cast<const float4_t*>(E0 + (chi * Ls + s) * Ls + 4 * kg);
    }
    sched_fence();
  };
  float acc[24];
#pragma unroll
  for (int k = 0; k < 24; ++k) acc[k] = 0.f;
  auto term = [&](auto kc) {
    constexpr int K = decltype(kc)::value;
    constexpr bool FWD = K % 2 == 0;
    constexpr int SIGN = (FWD ? -1 : 1) * (DAG ? -1 : 1);
    term_mfma<K / 2, SIGN, !FWD>(q[K].halves(0), q[K].halves(1), q[K].halves(2), lw[K], q[K].s, acc);
  };
  if (mask == 0xffu) {   // no branch between the loads: each term waits for its own
    static_for<8>([&](auto kc) {
      load_term(kc);
      sched_fence();
    });
    load_rest();
    static_for<8>([&](auto kc) {
      term(kc);
      pin24(acc);
    });
  } else {
    static_for<8>([&](auto kc) {
      if (mask >> decltype(kc)::value & 1) load_term(kc);
      sched_fence();
    });
    load_rest();
    static_for<8>([&](auto kc) {
      if (mask >> decltype(kc)::value & 1) term(kc);
      pin24(acc);
    });
  }

  // FP16 operands: every site scaled by its largest entry; the rows of the
  // centre field are first rounded over their own largest entry
  float rowmax = 0.f;
  uint32_t wp[12];
  if constexpr (HASW) {
    float v[24];
    wq.values(v);
#pragma unroll
    for (int k = 0; k < 24; ++k) rowmax = fmaxf(rowmax, fabsf(v[k]));
    const float im = rowmax > 0.f ? 1.f / rowmax : 0.f;
#pragma unroll
    for (int k = 0; k < 12; ++k) wp[k] = h2_bits(v[2 * k] * im, v[2 * k + 1] * im);
  }
  float cs = rowmax;
#pragma unroll
  for (int k = 0; k < 24; ++k) cs = fmaxf(cs, fabsf(acc[k]));
#pragma unroll
  for (int off = 1; off < Ls; off <<= 1) cs = fmaxf(cs, __shfl_xor(cs, off));
  const float ics = cs > 0.f ? 1.f / cs : 0.f;

  // tile: [site][component][slice]
  unsigned char* tile = tiles + wave * (NS * STR);
  uint16_t* mine = reinterpret_cast<uint16_t*>(tile + j * STR) + s;
  const unsigned char* rows = tile + ((col >> 2) + 4 * (g2 / NW)) * STR + (col & 3) * (2 * Ls) + 8 * kg;
  float4_t d[NG][6];   // a group's sums are valid in its own columns
#pragma unroll
  for (int i = 0; i < NG; ++i)
#pragma unroll
    for (int k = 0; k < 6; ++k) d[i][k] = float4_t{0.f, 0.f, 0.f, 0.f};
  auto product = [&](const uint32_t* w, const float4_t* m) {
#pragma unroll
    for (int k = 0; k < 12; ++k) {
      mine[2 * k * Ls] = (uint16_t)w[k];
      mine[(2 * k + 1) * Ls] = (uint16_t)(w[k] >> 16);
    }
    half4_t e[2];
#pragma unroll
    for (int chi = 0; chi < 2; ++chi)
#pragma unroll
      for (int v = 0; v < 4; ++v) e[chi][v] = (_Float16)m[chi][v];
    // the tile is the wavefront's own
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int k = 0; k < 6; ++k) {
      const u32x2 x = *reinterpret_cast<const u32x2*>(rows + 4 * k * (2 * Ls));
#pragma unroll
      for (int i = 0; i < NG; ++i) {
        const bool own = g2 / NW == i;
        const u32x2 a = {own ? x.x : 0u, own ? x.y : 0u};
        d[i][k] = __builtin_amdgcn_mfma_f32_16x16x16f16(__builtin_bit_cast(half4_t, a), e[k >= 3 ? 1 : 0], d[i][k], 0,
                                                        0, 0);
      }
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
  };
  uint32_t h[12];
#pragma unroll
  for (int k = 0; k < 12; ++k) h[k] = h2_bits(acc[2 * k] * ics, acc[2 * k + 1] * ics);
  product(h, m1);
  if constexpr (HASW) {
    if (live) {
      const float rsw = rowmax * ics;
#pragma unroll
      for (int k = 0; k < 12; ++k) h[k] = h2_bits(half_lo(wp[k]) * rsw, half_hi(wp[k]) * rsw);
      product(h, m0);
    }
  }
  float y[24];
#pragma unroll
  for (int k = 0; k < 24; ++k) {
    float v = d[0][k >> 2][k & 3];
#pragma unroll
    for (int i = 1; i < NG; ++i) v = col / Ls == i ? d[i][k >> 2][k & 3] : v;
    y[k] = v * cs;
  }
  Packed<S> pk;
  pk.from(y);
  const ChunkRsrc<S> ro(out);
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    if constexpr (std::is_same<S, __half>::value) __builtin_amdgcn_raw_buffer_store_b128(pk.q[k], ro.c[k], oo, 0, 0);
    else __builtin_amdgcn_raw_buffer_store_b64(pk.q[k], ro.c[k], oo, 0, 0);
  }
  __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(pk.s), ro.sc, ref.valid ? (uint32_t)ref.out5 * 4u : kAbsent, 0, 0);
  if constexpr (DOT) {
    if (dot_partial) {
      float pv[24], loc = 0.f;
      pq.values(pv);
#pragma unroll
      for (int k = 0; k < 24; ++k) loc += pv[k] * y[k];
      // the general kernel's order: a butterfly over the lanes (site, slice),
      // slice fastest, of each wavefront, then the wavefronts in turn; site
      // bits 0 and 1 are lane bits 4 and 5 here, further ones follow the slice
      double v = ref.valid ? (double)loc : 0.0;
      for (int off = 8; off >= Ls; off >>= 1) v += __shfl_xor(v, off);
      v += __shfl_xor(v, 32);
      v += __shfl_xor(v, 16);
      for (int off = Ls / 2; off > 0; off >>= 1) v += __shfl_xor(v, off);
      if (lane == 0) red[wave] = v;
      __syncthreads();
      if (threadIdx.x == 0) {
        double tot = 0;
        for (int i = 0; i < NW; ++i) tot += red[i];
        dot_partial[(int64_t)rhs * wk.nblk + blk] = tot;
      }
    }
  }
}

}  // namespace mspcg
