// Layout conversion between the canonical caller-facing arrays and the
// internal even-odd fields, and packing of the gauge links.
//
// Internal spinor half field (one parity): 5D site (i, s) where i is the
// site's index in the library's traversal order of that parity; the 24 reals
// of a site are interleaved complex, blocked over the Ls slices of a 4D site
// in chunks of 4 reals (RIRI), or split into 24 planes of length (V/2)*Ls
// ordered [re/im][spin][colour] (RRII); the offsets are in siteio.h.
// Links: [parity][mu][cb][18]
// (3x3 complex row-major, interleaved), with the boundary factor bc[mu]
// multiplied into U_mu(x) on the last slice x_mu = L_mu - 1, which is the one
// link used by both hops that cross that boundary.
#include "common.h"
#include "hopcore.h"
#include "siteio.h"

namespace qdwf {

namespace {

// One thread per (rhs, half, 5D site of that half).
template <class R, class S, int LAYOUT, bool UNPACK>
__global__ void pack_kernel(const void* __restrict__ src_v, void* __restrict__ dst_v, int nhalf,
                            int par0, long n5h, int Ls, int V, const int* __restrict__ site_lex,
                            int Vh, int nrhs) {
  const long total = (long)nrhs * nhalf * n5h;
  for (long idx = (long)blockIdx.x * blockDim.x + threadIdx.x; idx < total;
       idx += (long)gridDim.x * blockDim.x) {
    const long j = idx % n5h;
    const long rh = idx / n5h;
    const int h = (int)(rh % nhalf);
    const int r = (int)(rh / nhalf);
    const int p = par0 + h;
    const int cb = (int)(j / Ls), s = (int)(j % Ls);
    const int lex = site_lex[(long)p * Vh + cb];
    const long cidx = (((long)r * Ls + s) * V + lex) * 24;   // canonical reals
    const long ibase = ((long)r * nhalf + h) * n5h * 24;     // internal half field
    if (!UNPACK) {
      const R* src = reinterpret_cast<const R*>(src_v) + cidx;
      S* dst = reinterpret_cast<S*>(dst_v) + ibase;
#pragma unroll
      for (int c = 0; c < 24; ++c) {
        const S v = Store<S>::from64((double)src[c]);
        if (LAYOUT == QDWF_RIRI) dst[riri_offset(cb, s, c, Ls)] = v;
        else dst[rrii_offset(cb, s, c, Ls, n5h)] = v;
      }
    } else {
      const S* src = reinterpret_cast<const S*>(src_v) + ibase;
      R* dst = reinterpret_cast<R*>(dst_v) + cidx;
#pragma unroll
      for (int c = 0; c < 24; ++c) {
        const S v = (LAYOUT == QDWF_RIRI) ? src[riri_offset(cb, s, c, Ls)]
                                          : src[rrii_offset(cb, s, c, Ls, n5h)];
        dst[c] = (R)Store<S>::to(v);
      }
    }
  }
}

// Tiles of whole 4D sites through LDS, for the interleaved layout with Ls > 1:
// the canonical array keeps the 24 reals of one slice together and the slices
// a lattice apart, the internal one keeps the slices of a site together in
// chunks of 4 reals, so one lane per slice reads or writes scattered reals on
// one side. Here every access to memory is a 16-byte word of a contiguous run
// (24 reals of a slice; the Ls*24 reals of a site) and the transposition
// happens in LDS. Bound by memory: FP64 <-> complex128 at 16^3x32 x 16
// (0.81 GB moved) 230 -> 177 us, back 217 -> 170 us.
constexpr int kTileThreads = 256;
constexpr int kTileReals = 3072;   // reals of a tile at most (one site at least)

// n / d for n < 65536, d <= 65536, with m = div_magic(d)
__device__ __host__ inline uint32_t div_magic(uint32_t d) { return (uint32_t)(0x100000000ull / d) + 1u; }
__device__ inline int fast_div(int n, uint32_t m) { return (int)__umulhi((uint32_t)n, m); }

struct TileK {
  const void* src;
  void* dst;
  const int* site_lex;
  long n5h;
  int nhalf, par0, Ls, V, Vh;
  int ns_log2;            // sites per tile
  int ntile;              // tiles of a half field
  uint32_t m_ls, m_wps;   // division by Ls and by the 16-byte words of an internal site
  int nt;                 // store non-temporally (nt_stores)
};

template <class R, class S, bool UNPACK>
__global__ void __launch_bounds__(kTileThreads) pack_tile_kernel(TileK k) {
  constexpr int RW = 16 / (int)sizeof(R);      // reals of a canonical word
  constexpr int WPR = 24 / RW;                  // canonical words of a slice
  constexpr int E = 16 / (int)sizeof(S);        // reals of an internal word
  constexpr int ROW = 24 + RW;                  // LDS reals per slice (padded)
  extern __shared__ __align__(16) unsigned char smem[];
  R* t = reinterpret_cast<R*>(smem);            // [site][s][ROW]

  // logical block: parity fastest (the two parities of a region share the
  // canonical array's cache lines), then tiles, then right-hand sides
  const int B = xcd_remap(blockIdx.x, gridDim.x);
  const int h = B % k.nhalf;
  const int bt = B / k.nhalf;
  const int tile = bt % k.ntile;
  const long r = bt / k.ntile;
  const int ns = 1 << k.ns_log2, Ls = k.Ls;
  const int cb0 = tile << k.ns_log2;
  const int nsite = min(ns, k.Vh - cb0);
  const int* lex = k.site_lex + (long)(k.par0 + h) * k.Vh + cb0;
  const long canon = r * Ls * k.V;                                   // slices before this rhs
  const long ibase = (r * k.nhalf + h) * k.n5h * 24 + (long)cb0 * Ls * 24;
  const int ncw = WPR * Ls << k.ns_log2;        // canonical words of a full tile
  const int niw = nsite * (Ls * 24 / E);        // internal words of this tile

  auto canonical = [&](auto&& f) __attribute__((always_inline)) {
    for (int u = threadIdx.x; u < ncw; u += kTileThreads) {
      const int w = u % WPR, v = u / WPR;
      const int site = v & (ns - 1), s = v >> k.ns_log2;
      if (site < nsite)
        f((canon + (long)s * k.V + lex[site]) * 24 + w * RW, (site * Ls + s) * ROW + w * RW);
    }
  };
  auto internal = [&](auto&& f) __attribute__((always_inline)) {
    const int wps = Ls * 24 / E;
    for (int u = threadIdx.x; u < niw; u += kTileThreads) {
      const int site = fast_div(u, k.m_wps), w = u - site * wps;
      // the word's reals, two or four at a time: quad qd of the site is chunk
      // qd / Ls of slice qd % Ls
      int at[(E + 3) / 4];
#pragma unroll
      for (int j = 0; j < (E + 3) / 4; ++j) {
        const int e = w * E + 4 * j, qd = e >> 2;
        const int c = fast_div(qd, k.m_ls), s = qd - c * Ls;
        at[j] = (site * Ls + s) * ROW + c * 4 + (e & 3);
      }
      f(ibase + (long)u * E, at);
    }
  };

  if constexpr (!UNPACK) {
    const R* src = reinterpret_cast<const R*>(k.src);
    S* dst = reinterpret_cast<S*>(k.dst);
    canonical([&](long g, int l) {
      *reinterpret_cast<uint4*>(t + l) = *reinterpret_cast<const uint4*>(src + g);
    });
    __syncthreads();
    internal([&](long g, const int* at) {
      S v[E];
#pragma unroll
      for (int e = 0; e < E; ++e) v[e] = Store<S>::from64((double)t[at[e / 4] + e % 4]);
      uint4 w;
      __builtin_memcpy(&w, v, 16);
      uint4* o = reinterpret_cast<uint4*>(dst + g);
      if (k.nt) put_word<true>(o, w);
      else *o = w;
    });
  } else {
    const S* src = reinterpret_cast<const S*>(k.src);
    R* dst = reinterpret_cast<R*>(k.dst);
    internal([&](long g, const int* at) {
      const uint4 w = *reinterpret_cast<const uint4*>(src + g);
      S v[E];
      __builtin_memcpy(v, &w, 16);
#pragma unroll
      for (int e = 0; e < E; ++e) t[at[e / 4] + e % 4] = (R)Store<S>::to(v[e]);
    });
    __syncthreads();
    canonical([&](long g, int l) {
      const uint4 w = *reinterpret_cast<const uint4*>(t + l);
      uint4* o = reinterpret_cast<uint4*>(dst + g);
      if (k.nt) put_word<true>(o, w);
      else *o = w;
    });
  }
}

// Every precision of the links a context keeps, from one read of the
// canonical field: a block stages 64 links (consecutive sites of a parity,
// one direction; the boundary factor applied) in LDS and writes each
// precision's 64 x 18 reals, which are contiguous, in 16-byte words. One
// thread per link and one pass per precision wrote scattered reals instead:
// 16^3x32 from complex128, four precisions, 383 -> 49 us (0.23 GB moved).
constexpr int kLinkTile = 64;
struct LinkK {
  const void* U;
  void* out[4];           // per precision, nullptr where the context keeps none
  const int* site_lex;
  int Vh, V, L[4], bc[4], ntile;
};

template <class R>
__global__ void __launch_bounds__(256) link_tile_kernel(LinkK k) {
  constexpr int RW = 2;   // reals of a loaded word: one complex number
  __shared__ __align__(16) double t[kLinkTile * 18];
  __shared__ int lx[kLinkTile];
  __shared__ double fac[kLinkTile];
  // logical block: parity fastest, then directions, then tiles
  const int B = xcd_remap(blockIdx.x, gridDim.x);
  const int p = B & 1, mu = (B >> 1) & 3, tile = B >> 3;
  const int cb0 = tile * kLinkTile;
  const int n = min(kLinkTile, k.Vh - cb0);
  if ((int)threadIdx.x < n) {
    const int lex = k.site_lex[(long)p * k.Vh + cb0 + threadIdx.x];
    int rest = lex, c = 0;
    for (int m = 0; m <= mu; ++m) {
      c = rest % k.L[m];
      rest /= k.L[m];
    }
    lx[threadIdx.x] = lex;
    fac[threadIdx.x] = c == k.L[mu] - 1 ? (double)k.bc[mu] : 1.0;
  }
  __syncthreads();
  const R* U = reinterpret_cast<const R*>(k.U) + (long)mu * k.V * 18;
  for (int u = threadIdx.x; u < n * 9; u += 256) {
    const int l = u / 9, w = u - l * 9;
    const R* q = U + (long)lx[l] * 18 + w * RW;
    double a, b;
    if constexpr (sizeof(R) == 8) {
      const double2 v = *reinterpret_cast<const double2*>(q);
      a = v.x; b = v.y;
    } else {
      const float2 v = *reinterpret_cast<const float2*>(q);
      a = v.x; b = v.y;
    }
    t[l * 18 + w * 2] = fac[l] * a;
    t[l * 18 + w * 2 + 1] = fac[l] * b;
  }
  __syncthreads();
  const long base = (((long)p * 4 + mu) * k.Vh + cb0) * 18;
  auto put = [&](auto tag, void* out) {
    typedef decltype(tag) S;
    constexpr int E = 16 / (int)sizeof(S);
    if (!out) return;
    S* o = reinterpret_cast<S*>(out) + base;
    // 16-byte words while the tile is whole (its start is then aligned:
    // Vh * 18 reals and 64 * 18 reals are multiples of 16 bytes), else real by real
    if (n == kLinkTile && ((uintptr_t)o & 15) == 0) {
      for (int u = threadIdx.x; u < kLinkTile * 18 / E; u += 256) {
        S v[E];
#pragma unroll
        for (int e = 0; e < E; ++e) v[e] = Store<S>::from64(t[u * E + e]);
        uint4 w;
        __builtin_memcpy(&w, v, 16);
        reinterpret_cast<uint4*>(o)[u] = w;
      }
    } else {
      for (int u = threadIdx.x; u < n * 18; u += 256) o[u] = Store<S>::from64(t[u]);
    }
  };
  put(double(), k.out[QDWF_F64]);
  put(float(), k.out[QDWF_F32]);
  put(_Float16(), k.out[QDWF_F16]);
  put(bf16(), k.out[QDWF_BF16]);
}

template <class R, class S>
__global__ void link_kernel(const void* __restrict__ U_v, S* __restrict__ out, int Vh, int V,
                            const int* __restrict__ site_lex, int Lx, int Ly, int Lz, int Lt,
                            int bx, int by, int bz, int bt) {
  const long total = 2L * 4 * Vh;
  const R* U = reinterpret_cast<const R*>(U_v);
  for (long idx = (long)blockIdx.x * blockDim.x + threadIdx.x; idx < total;
       idx += (long)gridDim.x * blockDim.x) {
    const int cb = (int)(idx % Vh);
    const int mu = (int)((idx / Vh) % 4);
    const int p = (int)(idx / (4L * Vh));
    const int lex = site_lex[(long)p * Vh + cb];
    int c[4];
    int rest = lex;
    c[0] = rest % Lx; rest /= Lx;
    c[1] = rest % Ly; rest /= Ly;
    c[2] = rest % Lz;
    c[3] = rest / Lz;
    const int Lm[4] = {Lx, Ly, Lz, Lt};
    const int bm[4] = {bx, by, bz, bt};
    const double f = (c[mu] == Lm[mu] - 1) ? (double)bm[mu] : 1.0;
    const R* src = U + ((long)mu * V + lex) * 18;
    S* dst = out + idx * 18;
#pragma unroll
    for (int k = 0; k < 18; ++k) dst[k] = Store<S>::from64((double)f * (double)src[k]);
  }
}

inline int grid_for(long n) {
  long b = (n + 255) / 256;
  if (b > 65536) b = 65536;
  if (b < 1) b = 1;
  return (int)b;
}

}  // namespace

int launch_pack(qdwf_ctx* ctx, void* dst, int prec, int layout, const void* src, int src_prec,
                int subset, int nrhs, hipStream_t st, bool unpack) {
  const Geom& g = ctx->g;
  const int nhalf = (subset == QDWF_FULL) ? 2 : 1;
  const int par0 = (subset == QDWF_ODD) ? 1 : 0;
  const long total = (long)nrhs * nhalf * g.n5h;
  auto go = [&](auto rtag, auto stag) -> int {
    typedef decltype(rtag) R;
    typedef decltype(stag) S;
    // the tiled form where both arrays can be walked in 16-byte words; it
    // covers every Ls > 1 of the interleaved layout
    if (layout == QDWF_RIRI && g.Ls > 1 &&
        (((uintptr_t)src | (uintptr_t)dst) & 15) == 0) {
      TileK k;
      k.src = src;
      k.dst = dst;
      k.site_lex = ctx->d_site_lex;
      k.n5h = g.n5h;
      k.nhalf = nhalf; k.par0 = par0; k.Ls = g.Ls; k.V = g.V; k.Vh = g.Vh;
      k.ns_log2 = 0;
      while ((2 << k.ns_log2) * g.Ls * 24 <= kTileReals) ++k.ns_log2;
      k.ntile = (g.Vh + (1 << k.ns_log2) - 1) >> k.ns_log2;
      k.m_ls = div_magic((uint32_t)g.Ls);
      k.m_wps = div_magic((uint32_t)(g.Ls * 24 * sizeof(S) / 16));
      const long blocks = (long)k.ntile * nhalf * nrhs;
      if (blocks <= 0x7fffffffL) {
        // Stored non-temporally from 64 MiB (us, plain / non-temporal: pack FP16
        // from complex64 16^4 x 16 one parity, three right-hand sides, 76 / 64,
        // FP32 from complex128 12^3x24 x 12 the same 41 / 35), but a slice of a
        // complex64 field is 96 bytes: its lines reach memory in parts, the
        // other parity's sites between them (unpack 16^4 x 16 from FP32 27.2 /
        // 61.9, from FP16 19.6 / 58.5, three right-hand sides from FP64 191 /
        // 285). One parity from FP64 is bound by its reads and gains again
        // (24^4 x 8 137 / 103).
        const size_t bytes = (size_t)total * 24 * (unpack ? sizeof(R) : sizeof(S));
        const bool parts = unpack && sizeof(R) == 4 && (nhalf == 2 || sizeof(S) < 8);
        k.nt = !parts && bytes >= ((size_t)64 << 20);
        const size_t lds = ((size_t)g.Ls << k.ns_log2) * (24 * sizeof(R) + 16);
        if (unpack)
          hipLaunchKernelGGL((pack_tile_kernel<R, S, true>), dim3((unsigned)blocks),
                             dim3(kTileThreads), lds, st, k);
        else
          hipLaunchKernelGGL((pack_tile_kernel<R, S, false>), dim3((unsigned)blocks),
                             dim3(kTileThreads), lds, st, k);
        QDWF_HIP(hipGetLastError());
        return QDWF_OK;
      }
    }
    auto launch = [&](auto kern) {
      hipLaunchKernelGGL(kern, dim3(grid_for(total)), dim3(256), 0, st, src, dst, nhalf, par0,
                         g.n5h, g.Ls, g.V, ctx->d_site_lex, g.Vh, nrhs);
    };
    // pack reads canonical (src) and writes internal (dst); unpack the reverse
    if (!unpack) {
      if (layout == QDWF_RIRI) launch(pack_kernel<R, S, QDWF_RIRI, false>);
      else launch(pack_kernel<R, S, QDWF_RRII, false>);
    } else {
      if (layout == QDWF_RIRI) launch(pack_kernel<R, S, QDWF_RIRI, true>);
      else launch(pack_kernel<R, S, QDWF_RRII, true>);
    }
    QDWF_HIP(hipGetLastError());
    return QDWF_OK;
  };
  auto by_s = [&](auto rtag) -> int {
    switch (prec) {
      case QDWF_F64: return go(rtag, double());
      case QDWF_F32: return go(rtag, float());
      case QDWF_F16: return go(rtag, _Float16());
      case QDWF_BF16: return go(rtag, bf16());
    }
    return fail(QDWF_EINVAL, "unknown precision %d", prec);
  };
  if (src_prec == QDWF_F64) return by_s(double());
  if (src_prec == QDWF_F32) return by_s(float());
  return fail(QDWF_EINVAL, "canonical spinors are complex128 (QDWF_F64) or complex64 (QDWF_F32)");
}

int launch_pack_links(qdwf_ctx* ctx, const void* U, int canon_prec, hipStream_t st) {
  const Geom& g = ctx->g;
  const int* bc = ctx->act.bc;
  const long total = 2L * 4 * g.Vh;
  auto tiled = [&](auto rtag) -> int {
    typedef decltype(rtag) R;
    LinkK k;
    k.U = U;
    for (int p = 0; p < 4; ++p) k.out[p] = ctx->d_links[p];
    k.site_lex = ctx->d_site_lex;
    k.Vh = g.Vh;
    k.V = g.V;
    for (int mu = 0; mu < 4; ++mu) {
      k.L[mu] = g.L[mu];
      k.bc[mu] = bc[mu];
    }
    k.ntile = (g.Vh + kLinkTile - 1) / kLinkTile;
    hipLaunchKernelGGL((link_tile_kernel<R>), dim3((unsigned)k.ntile * 8), dim3(256), 0, st, k);
    QDWF_HIP(hipGetLastError());
    return QDWF_OK;
  };
  // a canonical complex number is loaded as one word: its alignment decides
  if (canon_prec == QDWF_F64 && ((uintptr_t)U & 15) == 0) return tiled(double());
  if (canon_prec == QDWF_F32 && ((uintptr_t)U & 7) == 0) return tiled(float());
  auto go = [&](auto rtag, auto stag, void* out) -> int {
    typedef decltype(rtag) R;
    typedef decltype(stag) S;
    if (!out) return QDWF_OK;   // a precision this context does not keep
    hipLaunchKernelGGL((link_kernel<R, S>), dim3(grid_for(total)), dim3(256), 0, st, U,
                       reinterpret_cast<S*>(out), g.Vh, g.V, ctx->d_site_lex, g.L[0], g.L[1],
                       g.L[2], g.L[3],
                       bc[0], bc[1], bc[2], bc[3]);
    QDWF_HIP(hipGetLastError());
    return QDWF_OK;
  };
  auto all = [&](auto rtag) -> int {
    int rc;
    if ((rc = go(rtag, double(), ctx->d_links[QDWF_F64]))) return rc;
    if ((rc = go(rtag, float(), ctx->d_links[QDWF_F32]))) return rc;
    if ((rc = go(rtag, _Float16(), ctx->d_links[QDWF_F16]))) return rc;
    return go(rtag, bf16(), ctx->d_links[QDWF_BF16]);
  };
  if (canon_prec == QDWF_F64) return all(double());
  if (canon_prec == QDWF_F32) return all(float());
  return fail(QDWF_EINVAL, "canonical gauge field is complex128 (QDWF_F64) or complex64 (QDWF_F32)");
}

}  // namespace qdwf
