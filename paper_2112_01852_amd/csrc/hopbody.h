// The Domain Wall kernel's body, shared by the launch over one context
// (hop.hip) and the grouped launch over many contexts (group.hip): the 4D
// Wilson hop D_h applied on every slice of the fifth dimension (the kernel
// Section 4.1 measures; 1320 flops per 5D site in Table 3), fused with the
// Mobius 5D factors and the 4D-local epilogue so that one pass over memory
// gives D, D^dag, M_pq, (M_qp)^dag, or the last stage of M_pc / M_pc^dag.
//
// Work decomposition (one lane per 5D site and right-hand side):
//   * a wavefront holds floor(64/Ls) groups of Ls lanes; the lanes of a group
//     are the Ls slices of one (4D site, rhs) pair, so the s +- 1 neighbours
//     needed by the 5D operator C live in the same wavefront and are fetched
//     with cross-lane permutes instead of memory reloads;
//   * a block covers nsb consecutive checkerboard sites times nrb right-hand
//     sides; the 8 links of each of its 4D sites (4 forward U_mu(x), 4 backward
//     U_mu(x-mu)) are staged once in LDS and shared by all Ls*nrb lanes of the
//     site (Section 4.2 credits the Domain Wall kernel's advantage over Wilson
//     Dslash to exactly this reuse of links across the fifth dimension);
//   * the spin projection (1 -+ g_mu) reduces each neighbour spinor to a
//     half spinor before the SU(3) multiply, so only 2 colour vectors are
//     multiplied per direction (Table 3 counts this as 1320 flops per site).
#pragma once

#include <type_traits>

#include "cgtypes.h"
#include "common.h"
#include "hopcore.h"
#include "pk16.h"
#include "siteio.h"
#include "spin.h"

namespace qdwf {

struct HopK {
  const void* in[2];
  void* out[2];
  const void* z[2];
  const void* links;   // [2][4][Vh][18] in the storage type
  const int* nbr;      // [2][8][Vh]
  long rs_in, rs_out, rs_z, plane;
  int Vh, Ls, nrhs, par0, npar;
  int nsb, nrb, gpw, nrblk;
  int epi, xcd, minv;
  double c_over_b, mf, hop_scale_b, alpha, beta;
  int nd, md;          // M_ee^-1 scan: Ls = 2^nd md, md odd
  double rpow[6];      // (-beta/alpha)^(2^j), j <= nd
  double rstep[4];     // (-beta/alpha)^(2^nd (m + 1)), m < md - 1
  const int* skip;     // per-rhs skip flags (HopArgs::skip), or nullptr
  int skip_stride;
  int cg;              // fused CG step (HopArgs::cg)
  void* cg_r;
  const double* cg_alpha;
  int cg_alpha_stride;
  double* cg_site;     // one sum per wavefront of each rhs
  int nw;              // wavefronts of a rhs: site_waves(Vh, Ls)
  void* cg_x;          // cg = 3: inner solution, compute type
  const void* cg_p;    // cg = 3: search direction, storage type
  int nt;              // store the output non-temporally (nt_stores)
  int split_off;       // SPLIT: byte offset of the half spinors in LDS
};

// Target occupancy (waves per SIMD) the register allocator plans for: two for
// 32- and 64-bit storage, whose arithmetic needs the registers to keep two
// directions' neighbour loads in flight (the FP32 launches of hop.hip take
// three instead); four for the packed FP16 path
// (interleaved layout, Ls = 16: neighbour spinors stay packed, 105-114
// registers, no spills), three for other 16-bit storage (BF16 at four: D
// 24^4 x 16 273 -> 277 us, D^dag 263 -> 272; the FP16 permute form spills 2-5
// registers at four, D 16^3x32 x 12 92.9 -> 89.6 but the solve at 12^4 x 12
// 16.04 -> 16.18 ms).
template <class S, int LAYOUT = QDWF_RRII, bool DPP16 = false> struct WavesPerEU {
  static constexpr int v =
      sizeof(S) >= 4 ? 2 : (std::is_same<S, _Float16>::value && LAYOUT == QDWF_RIRI && DPP16) ? 4 : 3;
};

// The 18 words of a link staged in LDS in its two sign-adjusted forms
// (link_words), read as four 16-byte and one 8-byte LDS loads.
__device__ inline void load_link_words(const float* p, uint32_t* U) {
  const uint4* q4 = reinterpret_cast<const uint4*>(p);
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const uint4 t4 = q4[j];
    U[4 * j] = t4.x; U[4 * j + 1] = t4.y; U[4 * j + 2] = t4.z; U[4 * j + 3] = t4.w;
  }
  const uint2 t2 = reinterpret_cast<const uint2*>(p)[8];
  U[16] = t2.x; U[17] = t2.y;
}

// One block's share of a hop launch: logical block L of the launch described
// by k (its sites, parity and right-hand sides), with smem the block's LDS
// (the LDS bytes make_hopk reports). Every 5D site's result depends only on
// k and the site, not on which block or launch computes it.
// CHI (D_h only, not the adjoint): without MINV the input already holds
// chi = (A/b) psi, so the hop takes it as it is; with MINV the result is
// multiplied by A/b after M_ee^-1 (the two commute: both are functions of
// C), so that the next hop of M_pc can take it as chi. MINV without CHI is
// for c = 0 (Shamir), where A/b = 1: nothing is applied before or after.
// FP16 storage in the interleaved layout takes the packed path (pk16.h):
// neighbour spinors stay packed, half spinors are projected in packed FP16
// and multiplied with v_dot2_f32_f16 into FP32. BF16 storage in that layout
// projects in FP32 and multiplies with v_dot2_f32_bf16 (no packed BF16 adds
// on this hardware).
//
// SPLIT (small launches): the four wavefronts of a block hold the same 64 / Ls
// sites, wavefront mu the two hops of direction mu; their partial sums meet
// in LDS and the first one carries on. A launch of fewer wavefronts than the
// chip has SIMDs takes as long as one wavefront does, and that is the latency
// of its loads: a lane alone waits for four pairs of neighbours one after
// another. (split_launch)
template <class S, int LAYOUT, bool DAG, bool DPP16, bool MINV, bool CHI = false, bool SPLIT = false>
__device__ inline void hop_block(const HopK& k, int L, unsigned char* smem) {
  typedef typename Store<S>::compute T;
  static_assert(!(DAG && CHI), "the adjoint hop applies A^dag once per site");
  constexpr bool PK = std::is_same<S, _Float16>::value && LAYOUT == QDWF_RIRI;
  // BF16 storage, interleaved: FP32 spinor arithmetic, SU(3) products as
  // v_dot2_f32_bf16 on the half spinor rounded to BF16 and the packed links
  constexpr bool PKB = std::is_same<S, bf16>::value && LAYOUT == QDWF_RIRI;
  constexpr int LSTR = LinkStride<T>::v;
  T* su = reinterpret_cast<T*>(smem);                       // [nsb][8][LSTR]
  int* snb = reinterpret_cast<int*>(su + (size_t)8 * LSTR * k.nsb);   // [8][nsb]

  // logical block L: parity fastest, then sites, then right-hand-side
  // blocks, so the right-hand sides sweep the lattice one after another and
  // the working set the caches see is one field at a time
  const int nsblk = (k.Vh + k.nsb - 1) / k.nsb;
  const int p = k.par0 + L % k.npar;
  const int t1 = L / k.npar;
  const int sb = t1 % nsblk;
  const int rb = t1 / nsblk;
  const int q = 1 - p;
  const int cb0 = sb * k.nsb;
  const int Vh = k.Vh;
  if (k.skip) {
    // the whole block returns (before any barrier) when none of its
    // right-hand sides is running
    bool run = false;
    for (int j = 0; j < k.nrb; ++j) {
      const int r = rb * k.nrb + j;
      if (r < k.nrhs && k.skip[(long)r * k.skip_stride] == 0) run = true;
    }
    if (!run) return;
  }

  // Stage the neighbour indices of the block's sites (one load per thread),
  // then start this lane's first two neighbour-spinor loads, then stage the
  // links with every load of this thread in flight at once, so the block pays
  // about two memory latencies before its arithmetic starts.
  const int* nbp = k.nbr + (long)p * 8 * Vh;
  for (int i = threadIdx.x; i < 8 * k.nsb; i += blockDim.x) {
    const int d = i / k.nsb, sl = i - d * k.nsb;
    const int cb = min(cb0 + sl, Vh - 1);
    snb[i] = nbp[(long)d * Vh + cb];
  }
  __syncthreads();

  const int Ls = DPP16 ? 16 : k.Ls;   // a constant on the Ls = 16 path
  const int lane = threadIdx.x & 63;
  const int mu0 = SPLIT ? __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)) : 0;
  const int wave = SPLIT ? 0 : (int)(threadIdx.x >> 6);   // among the wavefronts of the block's sites
  const int gl = lane / Ls, s = lane - gl * Ls;
  const bool lane_ok = gl < k.gpw;
  const int gid = wave * k.gpw + (lane_ok ? gl : 0);
  const int sl = gid / k.nrb, rl = gid - sl * k.nrb;
  const int cb = cb0 + sl, r = rb * k.nrb + rl;
  const bool active = lane_ok && cb < Vh && r < k.nrhs;
  const int rc = min(r, k.nrhs - 1);
  const int cbc = min(cb, Vh - 1);
  const S* in = reinterpret_cast<const S*>(k.in[p]) + (long)rc * k.rs_in;
  const int* nbs = snb + sl;

  // two neighbour spinors in flight (packed path: 12 words each)
  T va[24], vb[24];
  uint32_t wa[12], wb[12];
  // a site's 24 reals as 12 (re, im) FP16 words, in the order of SiteIO
  auto load_pk = [&](int site, uint32_t* w) {
    long i = site;
    int ss = s, lsb = Ls;
    riri_block(i, ss, lsb);
    const uint2* pp = reinterpret_cast<const uint2*>(in + i * lsb * 24 + (long)ss * 4);
#pragma unroll
    for (int c = 0; c < 6; ++c) {
      const uint2 qq = pp[c * lsb];
      w[2 * c] = qq.x;
      w[2 * c + 1] = qq.y;
    }
  };
  // (SPLIT: the wavefront's only two)
  const int n0 = SPLIT ? nbs[mu0 * k.nsb] : nbs[0], n1 = SPLIT ? nbs[(mu0 + 4) * k.nsb] : nbs[k.nsb];
  if constexpr (PK) {
    load_pk(n0, wa);
    load_pk(n1, wb);
  } else {
    SiteIO<S, LAYOUT>::load(in, n0, s, Ls, k.plane, va);
    SiteIO<S, LAYOUT>::load(in, n1, s, Ls, k.plane, vb);
  }

  {
    // one thread per link: 18 contiguous reals, loaded with vector loads
    // (packed path: 9 (re, im) words, staged in the two sign-adjusted forms
    // of link_words)
    const S* lk = reinterpret_cast<const S*>(k.links);
    const int nlink = 8 * k.nsb;
    for (int i = threadIdx.x; i < nlink; i += blockDim.x) {
      const int d = i / k.nsb, sl2 = i - d * k.nsb;
      const int mu = d & 3;
      int par, site;
      if (d < 4) { par = p; site = min(cb0 + sl2, Vh - 1); }
      else       { par = q; site = snb[d * k.nsb + sl2]; }
      const S* src = lk + (((long)par * 4 + mu) * Vh + site) * 18;
      if constexpr (PK || PKB) {
        const uint32_t* qw = reinterpret_cast<const uint32_t*>(src);
        uint32_t* dstw = reinterpret_cast<uint32_t*>(su + (sl2 * 8 + d) * LSTR);
        uint32_t w[9];
#pragma unroll
        for (int c = 0; c < 9; ++c) w[c] = qw[c];
#pragma unroll
        for (int c = 0; c < 9; ++c) link_words(w[c], d < 4, &dstw[c], &dstw[9 + c]);
      } else {
        T Ul[18];
        LinkIO<S>::load(src, Ul);
        T* dstp = su + (sl2 * 8 + d) * LSTR;
#pragma unroll
        for (int c = 0; c < 18; ++c) dstp[c] = Ul[c];
      }
    }
  }
  __syncthreads();

  const int base = gl * Ls;
  SShift<DPP16> sh;
  sh.src_m = lane_ok ? base + (s == 0 ? Ls - 1 : s - 1) : lane;   // holds slice s-1
  sh.src_p = lane_ok ? base + (s == Ls - 1 ? 0 : s + 1) : lane;   // holds slice s+1
  const T mf = (T)k.mf;
  const T wm = (s == 0) ? -mf : (T)1;        // wall factor of S_d at this slice
  const T wp = (s == Ls - 1) ? -mf : (T)1;   // wall factor of S_u at this slice
  // A = b (1 + (c/b) C); the factor b is applied once at the end
  const T cb_ = (T)k.c_over_b;
  const T cm = cb_ * wm, cp = cb_ * wp;
  const T* lks = su + sl * 8 * LSTR;
  // the same factors as FP16 pairs, for the packed path's A
  const uint32_t cmh = PK ? pk_f16((float)cm, (float)cm) : 0u;
  const uint32_t cph = PK ? pk_f16((float)cp, (float)cp) : 0u;

  T acc[24];
  // direction D uses the buffer loaded two steps earlier and refills it with
  // direction D + 2
  // (the link times the projected neighbour; its spin rows go into uh)
  auto hop_half = [&](auto Dc, T* uh) __attribute__((always_inline)) {
    constexpr int D = decltype(Dc)::value;
    constexpr int MU = D & 3;
    constexpr bool FWD = D < 4;
    // (1 - g) on forward hops and (1 + g) on backward ones; swapped for D_h^dag
    constexpr int SG = (FWD != DAG) ? -1 : +1;
    // chi / b = psi + (c/b) (P+ psi_{s-1} + P- psi_{s+1}), walls included,
    // unless the input already holds it (CHI without MINV, and always where
    // c = 0) or the hop is the adjoint's
    constexpr bool APPLY_A = !DAG && CHI == MINV;
    if constexpr (PK) {
      uint32_t* buf = (SPLIT ? !FWD : (D & 1)) ? wb : wa;
      uint32_t w[12];
#pragma unroll
      for (int i = 0; i < 12; ++i) w[i] = buf[i];
      if constexpr (!SPLIT && D < 6) load_pk(nbs[(D + 2) * k.nsb], buf);
      uint32_t h[6];
      if constexpr (APPLY_A) {
        // chi / b = psi + (c/b) (P+ psi_{s-1} + P- psi_{s+1}) in packed FP16:
        // upper spins (words 0-5) from slice s-1, lower (6-11) from s+1 (a
        // DPP row rotate at Ls = 16, a cross-lane permute otherwise)
        auto from_m = [&](uint32_t v) -> uint32_t {
          if constexpr (DPP16) return (uint32_t)dpp_ror<1>((int)v);
          else return (uint32_t)__shfl((int)v, sh.src_m, 64);
        };
        auto from_p = [&](uint32_t v) -> uint32_t {
          if constexpr (DPP16) return (uint32_t)dpp_ror<15>((int)v);
          else return (uint32_t)__shfl((int)v, sh.src_p, 64);
        };
        uint32_t x[12];
#pragma unroll
        for (int i = 0; i < 12; ++i)
          x[i] = i < 6 ? pk_fma(cmh, from_m(w[i]), w[i]) : pk_fma(cph, from_p(w[i]), w[i]);
        project_pk<MU, SG>(x, h);
      } else {
        project_pk<MU, SG>(w, h);
      }
      uint32_t U[18];
      load_link_words(lks + D * LSTR, U);
      su3_mul_pk<!FWD>(U, U + 9, h, uh);
    } else {
      T* buf = (SPLIT ? !FWD : (D & 1)) ? vb : va;
      T v[24];
#pragma unroll
      for (int i = 0; i < 24; ++i) v[i] = buf[i];
      if constexpr (!SPLIT && D < 6)
        SiteIO<S, LAYOUT>::load(in, nbs[(D + 2) * k.nsb], s, Ls, k.plane, buf);
      if constexpr (APPLY_A) {
        T w[24];
#pragma unroll
        for (int i = 0; i < 24; ++i) w[i] = v[i];
        shift_s<1, 15>(sh, cm, cp, w, v);
      }
      T h[12];
      project<MU, SG>(v, h);
      if constexpr (PKB) {
        uint32_t hw[6];
#pragma unroll
        for (int i = 0; i < 6; ++i) hw[i] = pk_bf16(h[2 * i], h[2 * i + 1]);
        uint32_t U[18];
        load_link_words(lks + D * LSTR, U);
        su3_mul_pk<!FWD, true>(U, U + 9, hw, uh);
      } else {
        T U[18];
        load_link(lks + D * LSTR, U);
        su3_mul<!FWD>(U, h, uh);
      }
    }
  };
  auto recon = [&](auto Dc, const T* uh) __attribute__((always_inline)) {
    constexpr int D = decltype(Dc)::value;
    constexpr int SG = ((D < 4) != DAG) ? -1 : +1;
    recon_acc<(D & 3), SG, D == 0>(uh, acc);
  };
  if constexpr (SPLIT) {
    T uf[12], ub[12];
    switch (mu0) {
      case 0: hop_half(IC<0>(), uf); hop_half(IC<4>(), ub); break;
      case 1: hop_half(IC<1>(), uf); hop_half(IC<5>(), ub); break;
      case 2: hop_half(IC<2>(), uf); hop_half(IC<6>(), ub); break;
      default: hop_half(IC<3>(), uf); hop_half(IC<7>(), ub); break;
    }
    // [6][12][64] half spinors behind the links and neighbour indices: the
    // forward and backward ones of mu = 1, 2, 3. The first wavefront adds all
    // eight in the order of the other form, so the two agree bit for bit.
    T* part = reinterpret_cast<T*>(smem + k.split_off) + lane;
    if (mu0 != 0) {
      T* o = part + (mu0 - 1) * 2 * 12 * 64;
#pragma unroll
      for (int i = 0; i < 12; ++i) {
        o[i * 64] = uf[i];
        o[(12 + i) * 64] = ub[i];
      }
    }
    __syncthreads();
    if (mu0 != 0) return;   // no barrier below
    auto add = [&](auto Dc) __attribute__((always_inline)) {
      constexpr int D = decltype(Dc)::value;
      T uh[12];
#pragma unroll
      for (int i = 0; i < 12; ++i) uh[i] = part[((((D & 3) - 1) * 2 + (D >> 2)) * 12 + i) * 64];
      recon(Dc, uh);
    };
    recon(IC<0>(), uf); add(IC<1>()); add(IC<2>()); add(IC<3>());
    recon(IC<4>(), ub); add(IC<5>()); add(IC<6>()); add(IC<7>());
  } else {
    auto step = [&](auto Dc) __attribute__((always_inline)) {
      T uh[12];
      hop_half(Dc, uh);
      recon(Dc, uh);
    };
    step(IC<0>()); step(IC<1>()); step(IC<2>()); step(IC<3>());
    step(IC<4>()); step(IC<5>()); step(IC<6>()); step(IC<7>());
  }

  if constexpr (DAG) {
    // A^dag h / b = h + (c/b) C^dag h, C^dag = P- S_d + P+ S_u:
    // upper spins come from s+1, lower spins from s-1
    T tmp[24];
#pragma unroll
    for (int i = 0; i < 24; ++i) tmp[i] = acc[i];
    shift_s<15, 1>(sh, cp, cm, acc, tmp);
#pragma unroll
    for (int i = 0; i < 24; ++i) acc[i] = tmp[i];
  }
  if constexpr (MINV) {
    // out = M_ee^-1 (or M_ee^-dag) applied to the hop result, across the
    // slices of the group: (alpha + beta S)^-1 on each chirality is a cyclic
    // geometric series in S, (1 / alpha) sum over k < Ls of rho^k S^k with
    // -mf on the terms that wrap; its common factor is folded into the scale.
    // M_ee: upper spins see S_d (slice s - d), lower spins S_u (s + d); the
    // adjoint swaps them.
    if constexpr (DPP16) {
      // summed by doubling (steps 1, 2, 4, 8)
      auto scan = [&](auto Jc) {
        constexpr int J = decltype(Jc)::value;
        constexpr int Dd = 1 << J;
        const T rp = (T)k.rpow[J];
        const T cdn = (s - Dd < 0) ? rp * (-mf) : rp;    // source slice s - d
        const T cup = (s + Dd >= 16) ? rp * (-mf) : rp;  // source slice s + d
        T src[24];
#pragma unroll
        for (int i = 0; i < 24; ++i) src[i] = acc[i];
        if constexpr (DAG) shift_s<16 - Dd, Dd>(sh, cup, cdn, src, acc);
        else shift_s<Dd, 16 - Dd>(sh, cdn, cup, src, acc);
      };
      scan(IC<0>()); scan(IC<1>()); scan(IC<2>()); scan(IC<3>());
    } else {
      // Ls = 2^nd md: nd doublings, then the md terms of step 2^nd at once,
      // the smallest first. With 32- and 64-bit storage the hop result (acc)
      // and the sum e of the series' other terms are kept apart and added once,
      // so that the leading part is rounded once and not in every doubling:
      // M_pc is then no further from the exact result than with the dense
      // inverse (in place, FP32 Moebius 1 % further: 8.14e-8 for 8.05e-8), for
      // 0.5 (FP64) to 1.5 % (FP32) of its time. 16-bit storage rounds far more.
      constexpr bool APART = sizeof(S) >= 4;
      T e[24];
#pragma unroll
      for (int i = 0; i < 24; ++i) e[i] = 0;
      auto shifted = [&](int d, T rp, T& cdn, T& cup, int& ldn, int& lup) __attribute__((always_inline)) {
        const int dn = s - d, up = s + d;
        cdn = dn < 0 ? rp * (-mf) : rp;
        cup = up >= Ls ? rp * (-mf) : rp;
        ldn = lane_ok ? base + (dn < 0 ? dn + Ls : dn) : lane;
        lup = lane_ok ? base + (up >= Ls ? up - Ls : up) : lane;
        if constexpr (DAG) {
          const T c = cdn; cdn = cup; cup = c;
          const int l = ldn; ldn = lup; lup = l;
        }
      };
      for (int j = 0; j < k.nd; ++j) {
        T cl, ch;
        int ll, lh;
        shifted(1 << j, (T)k.rpow[j], cl, ch, ll, lh);
#pragma unroll
        for (int i = 0; i < 24; ++i)
          if constexpr (APART)
            e[i] = fmac(i < 12 ? cl : ch, (T)__shfl(acc[i] + e[i], i < 12 ? ll : lh, 64), e[i]);
          else
            acc[i] = fmac(i < 12 ? cl : ch, (T)__shfl(acc[i], i < 12 ? ll : lh, 64), acc[i]);
      }
      if (k.md == 3) {
        // Ls = 12, 24 (and 6, 3): both terms of a component together
        T cl, ch, cl2, ch2;
        int ll, lh, ll2, lh2;
        shifted(1 << k.nd, (T)k.rstep[0], cl, ch, ll, lh);
        shifted(2 << k.nd, (T)k.rstep[1], cl2, ch2, ll2, lh2);
#pragma unroll
        for (int i = 0; i < 24; ++i) {
          const T v = APART ? acc[i] + e[i] : acc[i];
          e[i] = fmac(i < 12 ? cl : ch, (T)__shfl(v, i < 12 ? ll : lh, 64),
                      fmac(i < 12 ? cl2 : ch2, (T)__shfl(v, i < 12 ? ll2 : lh2, 64), e[i]));
        }
      } else if (k.md > 1) {
        // Ls = 10, 20 (md = 5) and 5
        T cl[4], ch[4];
        int ll[4], lh[4];
#pragma unroll
        for (int m = 0; m < 4; ++m) shifted((m + 1) << k.nd, (T)k.rstep[m], cl[m], ch[m], ll[m], lh[m]);
#pragma unroll
        for (int i = 0; i < 24; ++i) {
          const T v = APART ? acc[i] + e[i] : acc[i];
          T t = e[i];
#pragma unroll
          for (int m = 3; m >= 0; --m)
            t = fmac(i < 12 ? cl[m] : ch[m], (T)__shfl(v, i < 12 ? ll[m] : lh[m], 64), t);
          e[i] = t;
        }
      }
      if constexpr (APART && CHI) {
        T v[24];
#pragma unroll
        for (int i = 0; i < 24; ++i) v[i] = acc[i] + e[i];
        shift_s<1, 15>(sh, cm, cp, v, e);
      }
      if (APART || k.md > 1) {   // (in place, e holds the md terms alone)
#pragma unroll
        for (int i = 0; i < 24; ++i) acc[i] += e[i];
      }
    }
    if constexpr (CHI && (DPP16 || sizeof(S) < 4)) {
      // chi / b of the result for the next hop: (1 + (c/b) C) M_ee^-1 h
      T tmp[24];
#pragma unroll
      for (int i = 0; i < 24; ++i) tmp[i] = acc[i];
      shift_s<1, 15>(sh, cm, cp, tmp, acc);
    }
  }
  const T hs = (T)k.hop_scale_b;   // hop scale times b (and the M_ee^-1 factor)
  if (k.epi) {
    const S* zf = reinterpret_cast<const S*>(k.z[p]) + (long)rc * k.rs_z;
    T z[24];
    SiteIO<S, LAYOUT>::load(zf, cbc, s, Ls, k.plane, z);
    const T al = (T)k.alpha, be = (T)k.beta;
    const T bm = be * wm, bp = be * wp;
#pragma unroll
    for (int i = 0; i < 24; ++i) acc[i] = fmac(al, z[i], hs * acc[i]);
    if constexpr (!DAG) shift_s<1, 15>(sh, bm, bp, z, acc);   // + beta C z
    else shift_s<15, 1>(sh, bp, bm, z, acc);                  // + beta C^dag z
  } else {
#pragma unroll
    for (int i = 0; i < 24; ++i) acc[i] *= hs;
  }
  if (active && k.cg < 2) {
    S* out = reinterpret_cast<S*>(k.out[p]) + (long)rc * k.rs_out;
    if constexpr (PK) {
      long i = cbc;
      int ss = s, lsb = Ls;
      riri_block(i, ss, lsb);
      uint2* pp = reinterpret_cast<uint2*>(out + i * lsb * 24 + (long)ss * 4);
      uint2 w[6];
#pragma unroll
      for (int c = 0; c < 6; ++c)
        w[c] = make_uint2(pk_f16(acc[4 * c], acc[4 * c + 1]), pk_f16(acc[4 * c + 2], acc[4 * c + 3]));
      if (k.nt) {
#pragma unroll
        for (int c = 0; c < 6; ++c) put_word<true>(&pp[c * lsb], w[c]);
      } else {
#pragma unroll
        for (int c = 0; c < 6; ++c) pp[c * lsb] = w[c];
      }
    } else if (k.nt) {
      SiteIO<S, LAYOUT>::template store<true>(out, cbc, s, Ls, k.plane, acc);
    } else {
      SiteIO<S, LAYOUT>::store(out, cbc, s, Ls, k.plane, acc);
    }
  }
  if (!MINV && k.cg) {
    // the CG step: this 5D site's sum of squares (components in order), then
    // the sum over a wavefront's 5D sites by halves (FP64): wavefront w of a
    // right-hand side always holds checkerboard sites [w gpw, (w + 1) gpw),
    // so the sums do not depend on the launch shape. A site's sum is taken in
    // FP32 where the values are 16-bit numbers as stored (their squares are
    // exact in FP32, and 24 of them add with a relative error below 2^-19),
    // in FP64 otherwise. One value per wavefront is few enough for the next
    // launch to add in one block: per checkerboard site it took a reduction
    // launch more (4.5 us at any size, twice per iteration).
    const bool live = active && (!k.skip || k.skip[(long)rc * k.skip_stride] == 0);
    double ss = 0.0;
    if (k.cg == 1) {
      if constexpr (sizeof(S) == 2) {
        float s32 = 0.0f;
#pragma unroll
        for (int i = 0; i < 24; ++i) {
          const float v = (float)Store<S>::to(Store<S>::from(acc[i]));   // as stored
          s32 = __builtin_fmaf(v, v, s32);
        }
        ss = (double)s32;
      } else {
#pragma unroll
        for (int i = 0; i < 24; ++i) {
          const double v = (double)Store<S>::to(Store<S>::from(acc[i]));   // as stored
          ss += v * v;
        }
      }
    } else if (live) {
      typedef typename ResidStore<S>::t RS;
      RS* rr = reinterpret_cast<RS*>(k.cg_r) + (long)rc * k.rs_out;
      T rv[24];
      SiteIO<RS, LAYOUT>::load(rr, cbc, s, Ls, k.plane, rv);
      const T al = (T)k.cg_alpha[(long)rc * k.cg_alpha_stride];
      if constexpr (sizeof(RS) == 2) {
        float s32 = 0.0f;
#pragma unroll
        for (int i = 0; i < 24; ++i) {
          rv[i] = rv[i] - al * acc[i];
          const float v = (float)Store<RS>::to(Store<RS>::from(rv[i]));   // as stored
          s32 = __builtin_fmaf(v, v, s32);
        }
        ss = (double)s32;
      } else {
#pragma unroll
        for (int i = 0; i < 24; ++i) {
          rv[i] = rv[i] - al * acc[i];
          const double v = (double)Store<RS>::to(Store<RS>::from(rv[i]));   // as stored
          ss += v * v;
        }
      }
      if (k.nt) SiteIO<RS, LAYOUT>::template store<true>(rr, cbc, s, Ls, k.plane, rv);
      else SiteIO<RS, LAYOUT>::store(rr, cbc, s, Ls, k.plane, rv);
      if (k.cg == 3) {
        // the iteration's step at the same sites: x += alpha p
        T pv[24], xv[24];
        SiteIO<S, LAYOUT>::load(reinterpret_cast<const S*>(k.cg_p) + (long)rc * k.rs_out, cbc, s,
                                Ls, k.plane, pv);
        T* xr = reinterpret_cast<T*>(k.cg_x) + (long)rc * k.rs_out;
        SiteIO<T, LAYOUT>::load(xr, cbc, s, Ls, k.plane, xv);
#pragma unroll
        for (int i = 0; i < 24; ++i) xv[i] = xv[i] + al * pv[i];
        SiteIO<T, LAYOUT>::store(xr, cbc, s, Ls, k.plane, xv);
      }
    }
    double t = live ? ss : 0.0;
#pragma unroll
    for (int d = 32; d > 0; d >>= 1) t += __shfl_down(t, d, 64);
    const int w = SPLIT ? sb : sb * (int)(blockDim.x >> 6) + wave;
    if (lane == 0 && cb0 + wave * k.gpw < Vh) k.cg_site[(long)rc * k.nw + w] = t;
  }
}

// Ls = 2^nd md with md odd: the steps of the fused M_ee^-1.
inline void minv_steps(int Ls, int* nd, int* md) {
  *nd = 0;
  while (Ls % 2 == 0) {
    Ls /= 2;
    ++*nd;
  }
  *md = Ls;
}
// Whether the hop takes M_ee^-1 with it at this Ls: the series then costs at
// most seven shifts of the result (Ls = 8: 3, 12: 4, 16: 4, 20: 6, 24: 5, 32: 5,
// 40: 7, 48: 6), less than writing the hop's result and reading it in a launch
// of its own, also where one site leaves lanes of a wavefront idle
// (M_pc^dag M_pc 8^3x16, us, launch of its own / fused: Ls = 40 FP64 225 / 153,
// FP32 115 / 84, FP16 96 / 67; Ls = 48 456 / 164, 151 / 86, 124 / 66). Other
// Ls (odd factor 7 or more, and 64) keep launch_local.
inline bool minv_fused(int Ls) {
  int nd, md;
  minv_steps(Ls, &nd, &md);
  return md <= 5 && nd <= 5;
}

// Kernel arguments of a hop launch on one context (HopArgs as for
// launch_hop, the launch shape sh), its LDS bytes per block and its number of
// logical blocks. MINV: M_ee^-1 fused (minv_fused).
// split: for hop_block's SPLIT form (256 threads, one right-hand side per block).
template <class S, bool MINV>
int make_hopk(const qdwf_ctx* ctx, int prec, const HopArgs& a, const HopShape& sh, HopK* k,
              size_t* lds, int* nblocks, bool split = false) {
  typedef typename Store<S>::compute T;
  const Geom& g = ctx->g;
  for (int i = 0; i < 2; ++i) { k->in[i] = a.in[i]; k->out[i] = a.out[i]; k->z[i] = a.z[i]; }
  k->links = a.links ? a.links : ctx->d_links[prec];
  k->nbr = ctx->d_nbr;
  k->rs_in = a.rs_in; k->rs_out = a.rs_out; k->rs_z = a.rs_z;
  k->plane = g.n5h;
  k->Vh = g.Vh; k->Ls = g.Ls; k->nrhs = a.nrhs; k->par0 = a.par0; k->npar = a.npar;
  k->gpw = 64 / g.Ls;
  const int G = split ? k->gpw : (sh.threads / 64) * k->gpw;
  k->nrb = split ? 1 : sh.nrb;
  k->nsb = G / k->nrb;
  k->nrblk = (a.nrhs + k->nrb - 1) / k->nrb;
  const int nsblk = (g.Vh + k->nsb - 1) / k->nsb;
  k->epi = a.epi; k->xcd = sh.xcd;
  k->c_over_b = ctx->act.c / ctx->act.b;
  k->mf = ctx->act.mf;
  k->hop_scale_b = a.hop_scale * ctx->act.b;
  k->alpha = a.alpha; k->beta = a.beta;
  k->skip = a.skip;
  k->skip_stride = a.skip_stride;
  k->cg = a.cg;
  k->cg_r = a.cg_r;
  k->cg_alpha = a.cg_alpha;
  k->cg_alpha_stride = a.cg_alpha_stride;
  k->cg_site = a.cg_site;
  k->nw = site_waves(g.Vh, g.Ls);
  k->cg_x = a.cg_x;
  k->cg_p = a.cg_p;
  k->nt = nt_stores((size_t)a.npar * a.nrhs * g.n5h * 24 * sizeof(S), a.chained != 0, a.nrhs);
  if (a.cg && (a.cg > 3 || k->nrb != 1 || !a.epi || a.npar != 1 || !a.cg_site ||
               (a.cg >= 2 && (!a.cg_r || !a.cg_alpha)) || (a.cg == 3 && (!a.cg_x || !a.cg_p))))
    return fail(QDWF_EINVAL, "fused CG step needs a one-parity hop with epilogue and its buffers");
  k->minv = MINV;
  if (MINV) {
    if (a.epi) return fail(QDWF_EINVAL, "fused M_ee^-1 takes no epilogue term");
    if (!minv_fused(g.Ls)) return fail(QDWF_EINVAL, "fused M_ee^-1 does not take Ls = %d", g.Ls);
    const double al = ctx->act.b * (4.0 - ctx->act.M5) + 1.0;
    const double be = ctx->act.c * (4.0 - ctx->act.M5) - 1.0;
    minv_steps(g.Ls, &k->nd, &k->md);
    if (g.Ls == 16) {
      // the DPP form's own powers, by squaring
      double r = -be / al;
      for (int j = 0; j < 5; ++j) { k->rpow[j] = r; r *= r; }
      k->hop_scale_b /= al * (1.0 + ctx->act.mf * k->rpow[4]);
      k->rpow[5] = r;
    } else {
      // the inverse of M_ee as the hops apply it, every coefficient rounded
      // once: an error in one, the common factor above all, is in every value
      typedef long double LD;
      LD r = -(LD)be / al;
      for (int j = 0; j < 6; ++j) {
        k->rpow[j] = (double)r;
        if (j < k->nd) r *= r;
      }
      LD rs = 1;   // to (-beta/alpha)^Ls
      for (int m = 0; m < k->md; ++m) {
        rs *= r;
        if (m < 4) k->rstep[m] = (double)rs;
      }
      k->hop_scale_b = (double)((LD)a.hop_scale * ctx->act.b / (al * (1 + ctx->act.mf * rs)));
    }
  } else {
    k->nd = 0;
    k->md = 1;
    for (int j = 0; j < 6; ++j) k->rpow[j] = 0.0;
  }
  // links, neighbour table
  *lds = (size_t)8 * LinkStride<T>::v * k->nsb * sizeof(T) + (size_t)8 * k->nsb * sizeof(int) +
         (size_t)sh.lds_pad;
  k->split_off = 0;
  if (split) {
    k->split_off = (int)((*lds + 15) & ~(size_t)15);
    *lds = k->split_off + (size_t)6 * 12 * 64 * sizeof(T);
  }
  if (*lds > 64 * 1024) return fail(QDWF_EINVAL, "hop launch shape needs %zu bytes of LDS", *lds);
  *nblocks = nsblk * k->nrblk * a.npar;
  return QDWF_OK;
}

}  // namespace qdwf
