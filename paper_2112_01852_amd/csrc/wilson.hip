// The Wilson Dslash kernel (Section 4.1 names it beside the Domain Wall
// kernel; Table 1 measures it): the 4D hop D_h, optionally with the Wilson
// mass term, D_W = (4 + m) - D_h / 2.
//
// One lane per (5D site, rhs): for Ls = 1 a lane is one 4D site, for Ls > 1 the
// operator acts on every slice. Unlike the domain-wall kernel there is no
// reuse of links across the fifth dimension to exploit at Ls = 1, so each lane
// reads its 8 links straight from global memory and there is no LDS stage and
// no barrier. With Ls = 1 the links come from a lane-major copy built by
// qdwf_set_gauge: the 4 forward links of every site cut into chunks stored
// chunk-major over the sites, so that one load instruction of a wavefront
// reads consecutive words (5 loads per link instead of 9 narrow, strided
// ones); a backward link is read as its neighbour's forward link. With Ls > 1 the slices of a site
// share its links and the packed [parity][mu][site] links are read.
#include "common.h"
#include "hopcore.h"
#include "siteio.h"
#include "spin.h"

namespace qdwf {

namespace {

// Lane-major links of Ls = 1 contexts: for each parity and direction mu,
// four chunks of 4 reals, each chunk-major over the sites ([c][site][4]),
// then the last 2 reals of every link ([site][2]): 18 reals per link, no
// padding, and consecutive lanes read consecutive words. Forward links only:
// the backward link U_mu(x - mu) is the forward link of the neighbour.
template <class S> struct WLinkIO {
  typedef typename Store<S>::compute T;
  __device__ static inline void load(const S* __restrict__ w, int p, int mu, int i, int Vh, T* U) {
    const S* base = w + ((long)p * 4 + mu) * Vh * 18;
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      const S* q = base + ((long)c * Vh + i) * 4;
      if constexpr (sizeof(S) == 8) {
        const double2 a = reinterpret_cast<const double2*>(q)[0];
        const double2 b = reinterpret_cast<const double2*>(q)[1];
        U[4 * c] = (T)a.x; U[4 * c + 1] = (T)a.y; U[4 * c + 2] = (T)b.x; U[4 * c + 3] = (T)b.y;
      } else if constexpr (sizeof(S) == 4) {
        const float4 a = *reinterpret_cast<const float4*>(q);
        U[4 * c] = (T)a.x; U[4 * c + 1] = (T)a.y; U[4 * c + 2] = (T)a.z; U[4 * c + 3] = (T)a.w;
      } else {
        const uint2 a = *reinterpret_cast<const uint2*>(q);
        S h[4];
        __builtin_memcpy(h, &a, 8);
#pragma unroll
        for (int e = 0; e < 4; ++e) U[4 * c + e] = Store<S>::to(h[e]);
      }
    }
    const S* q = base + (long)Vh * 16 + (long)i * 2;
    if constexpr (sizeof(S) == 8) {
      const double2 a = *reinterpret_cast<const double2*>(q);
      U[16] = (T)a.x; U[17] = (T)a.y;
    } else if constexpr (sizeof(S) == 4) {
      const float2 a = *reinterpret_cast<const float2*>(q);
      U[16] = (T)a.x; U[17] = (T)a.y;
    } else {
      const uint32_t a = *reinterpret_cast<const uint32_t*>(q);
      S h[2];
      __builtin_memcpy(h, &a, 4);
      U[16] = Store<S>::to(h[0]); U[17] = Store<S>::to(h[1]);
    }
  }
};

struct WilK {
  const void* in[2];
  void* out[2];
  const void* z[2];
  const void* links;   // [2][4][Vh][18] in the storage type, boundary factors folded in
  const void* wl;      // Ls = 1: lane-major links (see WLinkIO), else null
  const int* nbr;      // [2][8][Vh]
  long rs_in, rs_out, rs_z, plane;
  int Vh, Ls, nrhs, par0, npar, epi;
  int nblk;            // blocks of one half field
  int nt;              // store the output non-temporally (nt_stores)
  double hop_scale, alpha;
};

// Launch form by storage type. The kernel is bound by what misses L2: the
// lanes in flight on an XCD at 16 waves per CU hold 12 MB of spinors and
// links in FP32, three times its L2, so a neighbour was gone again before the
// next direction asked for it. Fewer waves, each keeping the loads of the
// next directions in flight itself, move less (D_h at 32^3 x 64, us; the
// compiler's own occupancy and order, then this form): FP32 382 -> 256 at two
// waves per SIMD and two directions ahead (three ahead 256, one wave 282),
// FP64 733 -> 559 at one wave and two ahead (two waves spill: 693) in blocks
// of one wavefront (604 in blocks of four), FP16 195 -> 156 at two waves and
// three ahead (two ahead 165). That holds for FP16 on 4D fields (F4) in the
// interleaved layout. Elsewhere 16-bit storage runs at three waves and one
// ahead: BF16 unpacks what it prefetched at once and so holds 42 registers a
// direction, fields with Ls > 1 share a site's links between lanes, and split
// planes load reals singly (us, compiler's own / two waves, three ahead / this
// form: BF16 16^3x32 x 8 49.9 / 54.3 / 43.6, 12^4 x 12 13.8 / 15.7 / 14.4, 20^4 x
// 16 121 / 128 / 99, 4D 32^4 85 / 65 / 57, split planes 24^4 x 8 153 / 174 / 141;
// FP16 16^3x32 x 8 56.0 / 50.0 / 42.9, split planes 12^3x24 x 7 19.9 / 21.1 /
// 19.6; FP16 4D 32^4 interleaved 86 / 58.3 / 59.8, hence the exception).
template <class S, int LAYOUT, bool F4> struct WilsonForm {
  static constexpr bool narrow = sizeof(S) == 2;
  static constexpr bool deep = narrow && std::is_same<S, _Float16>::value && LAYOUT == QDWF_RIRI && F4;
  static constexpr int waves = sizeof(S) == 8 ? 1 : narrow && !deep ? 3 : 2;   // per SIMD
  static constexpr int ahead = deep ? 3 : narrow ? 1 : 2;                      // directions in flight
  static constexpr int threads = sizeof(S) == 8 ? 64 : 256;
};

// F4: 4D field; its links come lane-major where the type has such a copy (WL).
template <class S, int LAYOUT, bool DAG, bool F4, bool APART>
__global__ void __launch_bounds__((WilsonForm<S, LAYOUT, F4>::threads))
__attribute__((amdgpu_waves_per_eu((WilsonForm<S, LAYOUT, F4>::waves), (WilsonForm<S, LAYOUT, F4>::waves))))
wilson_kernel(WilK k) {
  typedef typename Store<S>::compute T;
  constexpr bool WL = F4 && sizeof(S) >= 4;
  constexpr int PD = WilsonForm<S, LAYOUT, F4>::ahead;
  const long n5 = (long)k.Vh * k.Ls;
  // logical block: parity fastest, then sites, then right-hand sides, each
  // XCD a contiguous range. Both parities of a region then run together and
  // read its links once from memory (before: 382 us, with this order alone
  // 323, FP32 at 32^3 x 64).
  // APART (run_wilson): the blocks of an XCD cover a contiguous range of sites
  // too, but one half field after another.
  int p, r, sb;
  if constexpr (APART) {
    int h;
    xcd_apart(blockIdx.x, gridDim.x, k.npar * k.nrhs, &h, &sb);
    p = k.par0 + (k.npar == 2 ? h & 1 : 0);
    r = k.npar == 2 ? h >> 1 : h;
  } else {
    const int B = xcd_remap(blockIdx.x, gridDim.x);
    p = k.par0 + B % k.npar;
    sb = B / k.npar;
    r = sb / k.nblk;
    sb -= r * k.nblk;
  }
  const long j = (long)sb * blockDim.x + threadIdx.x;
  if (j >= n5) return;   // no barrier below
  const int q = 1 - p;
  const int i = (int)(j / k.Ls), s = (int)(j - (long)i * k.Ls);
  const int Vh = k.Vh;
  const S* in = reinterpret_cast<const S*>(k.in[p]) + (long)r * k.rs_in;
  const S* lk = reinterpret_cast<const S*>(k.links);
  const int* nb = k.nbr + (long)p * 8 * Vh;

  int nn[8];
#pragma unroll
  for (int d = 0; d < 8; ++d) nn[d] = nb[(long)d * Vh + i];
  // spinor and link of directions D .. D + PD - 1, in buffers D % PD
  T vb[PD][24], ub[PD][18];
  auto fetch = [&](auto Dc) __attribute__((always_inline)) {
    constexpr int D = decltype(Dc)::value;
    if constexpr (D < 8) {
      constexpr int MU = D & 3;
      constexpr bool FWD = D < 4;
      const int n = nn[D];
      SiteIO<S, LAYOUT>::load(in, n, s, k.Ls, k.plane, vb[D % PD]);
      // forward: U_mu(x) of this site; backward: U_mu(x - mu) of the neighbour
      if constexpr (WL) {
        WLinkIO<S>::load(reinterpret_cast<const S*>(k.wl), FWD ? p : q, MU, FWD ? i : n, Vh,
                         ub[D % PD]);
      } else {
        const long li = FWD ? (((long)p * 4 + MU) * Vh + i) : (((long)q * 4 + MU) * Vh + n);
        LinkIO<S>::load(lk + li * 18, ub[D % PD]);
      }
    }
  };
  T acc[24];
  auto step = [&](auto Dc) __attribute__((always_inline)) {
    constexpr int D = decltype(Dc)::value;
    constexpr int MU = D & 3;
    constexpr bool FWD = D < 4;
    // (1 - g) on forward hops and (1 + g) on backward ones; swapped for D_h^dag
    constexpr int SG = (FWD != DAG) ? -1 : +1;
    T U[18], h[12], uh[12];
    project<MU, SG>(vb[D % PD], h);
#pragma unroll
    for (int c = 0; c < 18; ++c) U[c] = ub[D % PD][c];
    fetch(IC<D + PD>());
    su3_mul<!FWD>(U, h, uh);
    recon_acc<MU, SG, D == 0>(uh, acc);
  };
  fetch(IC<0>());
  if constexpr (PD > 1) fetch(IC<1>());
  if constexpr (PD > 2) fetch(IC<2>());
  step(IC<0>()); step(IC<1>()); step(IC<2>()); step(IC<3>());
  step(IC<4>()); step(IC<5>()); step(IC<6>()); step(IC<7>());

  const T hs = (T)k.hop_scale;
  if (k.epi) {
    const S* zf = reinterpret_cast<const S*>(k.z[p]) + (long)r * k.rs_z;
    T z[24];
    SiteIO<S, LAYOUT>::load(zf, i, s, k.Ls, k.plane, z);
    const T al = (T)k.alpha;
#pragma unroll
    for (int c = 0; c < 24; ++c) acc[c] = fmac(al, z[c], hs * acc[c]);
  } else {
#pragma unroll
    for (int c = 0; c < 24; ++c) acc[c] *= hs;
  }
  S* out = reinterpret_cast<S*>(k.out[p]) + (long)r * k.rs_out;
  if (k.nt) SiteIO<S, LAYOUT>::template store<true>(out, i, s, k.Ls, k.plane, acc);
  else SiteIO<S, LAYOUT>::store(out, i, s, k.Ls, k.plane, acc);
}

template <class S, int LAYOUT, bool DAG>
int run_wilson(qdwf_ctx* ctx, int prec, const HopArgs& a, hipStream_t st) {
  const Geom& g = ctx->g;
  WilK k;
  for (int h = 0; h < 2; ++h) { k.in[h] = a.in[h]; k.out[h] = a.out[h]; k.z[h] = a.z[h]; }
  k.links = ctx->d_links[prec];
  k.wl = (g.Ls == 1) ? ctx->d_wlinks[prec] : nullptr;
  k.nbr = ctx->d_nbr;
  k.rs_in = a.rs_in; k.rs_out = a.rs_out; k.rs_z = a.rs_z;
  k.plane = g.n5h;
  k.Vh = g.Vh; k.Ls = g.Ls; k.nrhs = a.nrhs; k.par0 = a.par0; k.npar = a.npar;
  k.epi = a.epi;
  k.hop_scale = a.hop_scale;
  k.alpha = a.alpha;
  constexpr int NT = WilsonForm<S, LAYOUT, true>::threads;   // whether 4D or not
  const long nblk = (g.n5h + NT - 1) / NT;
  const long blocks = nblk * a.npar * a.nrhs;
  k.nt = nt_stores((size_t)a.npar * a.nrhs * g.n5h * 24 * sizeof(S), a.chained != 0, a.nrhs);
  k.nblk = (int)nblk;
  if (blocks > 0x7fffffffL) return fail(QDWF_EINVAL, "problem too large for one launch");
  // One half field after another (APART) while an XCD still finds in the
  // caches what half fields share, their links: its neighbouring blocks then
  // share spinors too. D_h, us, half field fastest / apart: FP32 16^3x32 17.7 /
  // 16.6, 20^4 24.1 / 22.1, 16^3x48 25.3 / 25.1; FP64 16^3x32 37.6 / 36.5;
  // batches FP32 16^4 with 2, 4 and 12 right-hand sides 17.6 / 15.2, 30.3 /
  // 25.6, 82 / 69, of one parity 9.1 / 7.7, 16.3 / 11.7, 43 / 30, FP64 with 12
  // 190 / 175, FP16 20^4 of one parity with 4 23.6 / 21.8. Past the lines: FP32
  // 16^2x32^2 33.4 / 33.9, 32^3x64 255 / 328, of one parity 16^3x32 with 4 31.5
  // / 31.8, 20^4 with 4 37.6 / 39.4. A single 16-bit field does not gain (FP16
  // 20^4 15.3 / 15.7), and with Ls > 1 the slices share the links already.
  const long lanes = 2 * g.n5h;   // of one right-hand side, both parities
  const bool apart = g.Ls == 1 && a.npar * a.nrhs > 1 &&
                     (a.nrhs == 1 ? sizeof(S) >= 4 && lanes <= 196608
                                  : lanes <= (sizeof(S) >= 4 ? 98304 : 196608));
  auto launch = [&](auto kern) {
    hipLaunchKernelGGL(kern, dim3((unsigned)blocks), dim3(NT), 0, st, k);
  };
  if (sizeof(S) >= 4 ? k.wl != nullptr : g.Ls == 1) {
    if (apart) launch(wilson_kernel<S, LAYOUT, DAG, true, true>);
    else launch(wilson_kernel<S, LAYOUT, DAG, true, false>);
  } else {
    if (apart) launch(wilson_kernel<S, LAYOUT, DAG, false, true>);
    else launch(wilson_kernel<S, LAYOUT, DAG, false, false>);
  }
  QDWF_HIP(hipGetLastError());
  return QDWF_OK;
}

template <class S>
__global__ void wlink_kernel(const S* __restrict__ links, S* __restrict__ wl, int Vh) {
  const long total = 2L * 4 * Vh;
  for (long t = (long)blockIdx.x * blockDim.x + threadIdx.x; t < total;
       t += (long)gridDim.x * blockDim.x) {
    const int i = (int)(t % Vh);
    const long pm = t / Vh;   // parity * 4 + mu, as in the packed links
    const S* src = links + t * 18;
    S* base = wl + pm * Vh * 18;
#pragma unroll
    for (int c = 0; c < 4; ++c)
#pragma unroll
      for (int e = 0; e < 4; ++e) base[((long)c * Vh + i) * 4 + e] = src[4 * c + e];
    base[(long)Vh * 16 + (long)i * 2] = src[16];
    base[(long)Vh * 16 + (long)i * 2 + 1] = src[17];
  }
}

}  // namespace

int launch_wilson_links(qdwf_ctx* ctx, hipStream_t st) {
  const Geom& g = ctx->g;
  const long total = 2L * 4 * g.Vh;
  long blocks = (total + 255) / 256;
  if (blocks > 65536) blocks = 65536;
  auto go = [&](auto tag, int p) {
    typedef decltype(tag) S;
    hipLaunchKernelGGL(wlink_kernel<S>, dim3((unsigned)blocks), dim3(256), 0, st,
                       reinterpret_cast<const S*>(ctx->d_links[p]),
                       reinterpret_cast<S*>(ctx->d_wlinks[p]), g.Vh);
  };
  for (int p = QDWF_F64; p <= QDWF_BF16; ++p) {
    if (!ctx->d_wlinks[p]) continue;
    if (p == QDWF_F64) go(double(), p);
    else if (p == QDWF_F32) go(float(), p);
    else if (p == QDWF_F16) go(_Float16(), p);
    else go(bf16(), p);
    QDWF_HIP(hipGetLastError());
  }
  return QDWF_OK;
}

int launch_wilson(qdwf_ctx* ctx, int prec, int layout, int dagger, const HopArgs& a,
                  hipStream_t st) {
  auto go = [&](auto tag_s) -> int {
    typedef decltype(tag_s) S;
    if (layout == QDWF_RIRI)
      return dagger ? run_wilson<S, QDWF_RIRI, true>(ctx, prec, a, st)
                    : run_wilson<S, QDWF_RIRI, false>(ctx, prec, a, st);
    return dagger ? run_wilson<S, QDWF_RRII, true>(ctx, prec, a, st)
                  : run_wilson<S, QDWF_RRII, false>(ctx, prec, a, st);
  };
  switch (prec) {
    case QDWF_F64: return go(double());
    case QDWF_F32: return go(float());
    case QDWF_F16: return go(_Float16());
    case QDWF_BF16: return go(bf16());
  }
  return fail(QDWF_EINVAL, "unknown precision %d", prec);
}

}  // namespace qdwf
