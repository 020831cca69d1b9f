// The Domain Wall kernel launched over one context: the 4D Wilson hop D_h on
// every slice of the fifth dimension fused with the Mobius 5D factors and the
// 4D-local epilogue (the body and its work decomposition are in hopbody.h).
#include <cstdlib>
#include <type_traits>

#include "hopbody.h"

namespace qdwf {

namespace {

// Waves per SIMD of a launch: FP32 in the interleaved layout runs at three
// (129-138 registers, no spills), which measured faster than two for the
// one-parity hops (2-4 %) and, since outputs are stored non-temporally, for
// the full operator too (D 16^3x32 x 8 93.0 -> 86.2 us, 16^4 x 12 73.0 ->
// 65.3, 24^4 x 16 355 -> 349; D^dag 84.1 -> 80.2, 63.6 -> 59.8, 349 -> 342).
template <class S, int LAYOUT, bool DPP16> struct HopWaves {
  static constexpr int v = (std::is_same<S, float>::value && LAYOUT == QDWF_RIRI)
                               ? 3 : WavesPerEU<S, LAYOUT, DPP16>::v;
};

template <class S, int LAYOUT, bool DAG, bool DPP16, bool MINV, bool CHI>
__global__ void __launch_bounds__(256)
__attribute__((amdgpu_waves_per_eu(HopWaves<S, LAYOUT, DPP16>::v,
                                   HopWaves<S, LAYOUT, DPP16>::v)))
hop_kernel(HopK k) {
  extern __shared__ __align__(16) unsigned char smem[];
  // the XCD remap hands each XCD a contiguous range of logical blocks
  const int L = k.xcd ? xcd_remap(blockIdx.x, gridDim.x) : (int)blockIdx.x;
  hop_block<S, LAYOUT, DAG, DPP16, MINV, CHI>(k, L, smem);
}

// Small launches in the interleaved layout (hop_block's SPLIT form).
template <class S, bool DAG, bool DPP16, bool MINV, bool CHI>
__global__ void __launch_bounds__(256)
__attribute__((amdgpu_waves_per_eu(sizeof(S) == 8 ? 1 : 2, sizeof(S) == 8 ? 1 : 2)))
hop_split_kernel(HopK k) {
  extern __shared__ __align__(16) unsigned char smem[];
  hop_block<S, QDWF_RIRI, DAG, DPP16, MINV, CHI, true>(k, blockIdx.x, smem);
}

// Whether a launch takes the SPLIT form: while four wavefronts for each of
// the launch's own have room on the chip's 1024 SIMDs at once, at one (FP64)
// or two per SIMD, and the half spinors fit LDS beside the shape's padding.
// us, 256-thread blocks / one wavefront a block / SPLIT: FP64 D 4^4 x 8 12.0 /
// 9.1 / 8.1 (8 is what the call costs the host), M_pc^dag M_pc FP64 4^4 x 16
// 36.0 / 27.9 / 25.1, FP32 8^4 x 8 34.7 / 30.7 / 26.4, FP16 8^4 x 16 (512
// wavefronts) 27.5 / 25.4 / 24.5; past the line FP64 8^4 x 16 44.4 / 37.4 /
// 55.2, FP16 D 8^4 x 16 (1024 wavefronts) 8.1 / 8.0 / 10.3.
template <class S> bool split_launch(const qdwf_ctx* ctx, const HopArgs& a, const HopShape& sh) {
  if (!sh.split) return false;
  typedef typename Store<S>::compute T;
  const int gpw = 64 / ctx->g.Ls;
  const size_t lds = (size_t)gpw * 8 * (LinkStride<T>::v * sizeof(T) + sizeof(int)) + 16 +
                     (size_t)sh.lds_pad + (size_t)6 * 12 * 64 * sizeof(T);
  return lds <= 64 * 1024 && (long)site_waves(ctx->g.Vh, ctx->g.Ls) * a.npar * a.nrhs <=
                                 (sizeof(S) == 8 ? 256 : 512);
}

template <class S, int LAYOUT, bool DAG, bool DPP16, bool MINV, bool CHI>
int run_hop_k(qdwf_ctx* ctx, int prec, const HopArgs& a, hipStream_t st, const HopShape& sh) {
  HopK k;
  size_t lds = 0;
  int nb = 0;
  if constexpr (LAYOUT == QDWF_RIRI) {
    if (split_launch<S>(ctx, a, sh)) {
      int rc = make_hopk<S, MINV>(ctx, prec, a, sh, &k, &lds, &nb, true);
      if (rc) return rc;
      hipLaunchKernelGGL((hop_split_kernel<S, DAG, DPP16, MINV, CHI>), dim3(nb), dim3(256), lds, st, k);
      QDWF_HIP(hipGetLastError());
      return QDWF_OK;
    }
  }
  int rc = make_hopk<S, MINV>(ctx, prec, a, sh, &k, &lds, &nb);
  if (rc) return rc;
  hipLaunchKernelGGL((hop_kernel<S, LAYOUT, DAG, DPP16, MINV, CHI>), dim3(nb), dim3(sh.threads), lds,
                     st, k);
  QDWF_HIP(hipGetLastError());
  return QDWF_OK;
}

template <class S, int LAYOUT, bool DAG>
int run_hop(qdwf_ctx* ctx, int prec, const HopArgs& a, hipStream_t st, const HopShape& sh) {
  if (a.chi && DAG) return fail(QDWF_EINVAL, "the adjoint hop takes no A-applied input");
  if constexpr (!DAG) {
    if (a.chi) {
      if (ctx->g.Ls == 16)
        return a.minv ? run_hop_k<S, LAYOUT, false, true, true, true>(ctx, prec, a, st, sh)
                      : run_hop_k<S, LAYOUT, false, true, false, true>(ctx, prec, a, st, sh);
      return a.minv ? run_hop_k<S, LAYOUT, false, false, true, true>(ctx, prec, a, st, sh)
                    : run_hop_k<S, LAYOUT, false, false, false, true>(ctx, prec, a, st, sh);
    }
  }
  if (ctx->g.Ls == 16)
    return a.minv ? run_hop_k<S, LAYOUT, DAG, true, true, false>(ctx, prec, a, st, sh)
                  : run_hop_k<S, LAYOUT, DAG, true, false, false>(ctx, prec, a, st, sh);
  return a.minv ? run_hop_k<S, LAYOUT, DAG, false, true, false>(ctx, prec, a, st, sh)
                : run_hop_k<S, LAYOUT, DAG, false, false, false>(ctx, prec, a, st, sh);
}

}  // namespace

// Wavefronts of a launch (of one parity) up to which blocks have one wavefront.
constexpr long kSmallWaves = 4096;

bool hop_splits(const qdwf_ctx* ctx, int prec, int layout, const HopArgs& a, const HopShape& sh) {
  if (layout != QDWF_RIRI) return false;
  switch (prec) {
    case QDWF_F64: return split_launch<double>(ctx, a, sh);
    case QDWF_F32: return split_launch<float>(ctx, a, sh);
    case QDWF_F16: return split_launch<_Float16>(ctx, a, sh);
  }
  return split_launch<bf16>(ctx, a, sh);
}

HopShape default_shape(const qdwf_ctx* ctx, int prec, int nrhs) {
  HopShape sh;
  // at most 32 (site, rhs) groups per block: bounds the LDS link stage
  // (32 sites x 8 links x 18 reals, 36 KB in FP64) for every Ls
  const int gpw = 64 / ctx->g.Ls;
  int waves = 32 / gpw;
  if (waves < 1) waves = 1;
  if (waves > 4) waves = 4;
  sh.threads = 64 * waves;
  // small launches in blocks of one wavefront, which reach more CUs. us, blocks
  // of four / of one: M_pc^dag M_pc FP64 8^4 x 16 (512 wavefronts of a parity)
  // 44.4 / 37.4, FP16 12^4 x 16 (2592) 44.7 / 42.6, 12^3x16 (3456) 52.0 / 50.3,
  // 12^3x24 (5184) 71.7 / 68.4, 16^3x32 (16384) 172.7 / 171.2; FP32 3456 80.1 /
  // 80.6, 5184 118 / 116, 16384 292 / 298; FP64 2592 130.2 / 130.4, 5184 260 /
  // 256, 16384 612 / 637. FP64 D is the one with a loss below the line, at Ls =
  // 16 (3456: 76.6 / 79.1) though not at Ls = 8 (2592: 69.0 / 66.4).
  if ((long)site_waves(ctx->g.Vh, ctx->g.Ls) * nrhs <= kSmallWaves) sh.threads = 64;
  sh.split = 1;
  sh.xcd = 1;
  // one right-hand side per block: with the right-hand sides outermost in the
  // block order this measured faster than sharing the staged links between
  // several right-hand sides of a block (the tuner still tries both)
  sh.nrb = 1;
  sh.lds_pad = 0;
  // the t-sweep of the full operator, in FP32 with 16- and 32-wide rows (one
  // and two blocks of 8 waves per CU): us, sweep / checkerboard, D 32^4 x 16
  // 991 / 1064, 16^3x64 259 / 268, 16x24^3 223 / 227. Since the checkerboard
  // kernel streams its outputs it is the faster one on small lattices (16^4
  // 65 / 56, 16^3x32 120 / 102, 32x16^3 131 / 104, c = 0 alike), which the tuner
  // finds. Slower with 24-wide rows (6 waves per CU), in BF16 storage, and in
  // FP16 storage since the checkerboard kernel keeps FP16 neighbours packed
  // (32^4 x 16 D 0.73 against 0.84 ms); the tuner tries it wherever it applies
  const int Lx = ctx->g.L[0];
  sh.sweep = (prec == QDWF_F32 && (Lx == 16 || Lx == 32)) ? 1 : 0;
  if (const char* e = std::getenv("QDWF_HOP_LDS_PAD")) sh.lds_pad = std::atoi(e);
  if (const char* e = std::getenv("QDWF_HOP_THREADS")) {
    const int t = std::atoi(e);
    if (t >= 64 && t <= 256 && t % 64 == 0) {
      sh.threads = t;
      sh.split = 0;
    }
  }
  return sh;
}

int launch_hop(qdwf_ctx* ctx, int prec, int layout, int dagger, const HopArgs& a0,
               hipStream_t st, const HopShape* shape) {
  HopArgs a = a0;
  // Shamir (c = 0): A/b = 1, so every input is its own chi and no neighbour
  // goes through the s +- 1 exchange (us: D FP64 16^3x32 x 8 180 -> 166, FP32
  // 93 -> 79, FP16 54 -> 42; M_pc^dag M_pc FP64 16^4 x 8 193 -> 184)
  if (!dagger && ctx->act.c == 0.0) a.chi = a.minv ? 0 : 1;
  else if (!dagger && a.minv && !a.chi) return fail(QDWF_EINVAL, "fused M_ee^-1 hands on A/b times its result");
  HopShape sh;
  if (shape) sh = *shape;
  else if (!tuned_shape(ctx, prec, layout, dagger, a.nrhs, &sh)) sh = default_shape(ctx, prec, a.nrhs);
  // the fused CG step sums one right-hand side per wavefront
  if (a.cg && sh.nrb != 1) sh = default_shape(ctx, prec, a.nrhs);
  const int G = (sh.threads / 64) * (64 / ctx->g.Ls);
  if (sh.threads % 64 || sh.threads < 64 || sh.threads > 256 || sh.nrb < 1 || G % sh.nrb)
    return fail(QDWF_EINVAL, "invalid hop launch shape (threads %d, nrb %d)", sh.threads, sh.nrb);
  // the full operator on one whole field takes the t-sweep where it applies
  // (QDWF_SWEEP=1 / 0 forces it on / off where it applies)
  const char* force = std::getenv("QDWF_SWEEP");
  const bool sweep = (force && *force) ? force[0] == '1' : sh.sweep != 0;
  if (sweep && sweep_eligible(ctx, prec, layout, a)) return launch_sweep(ctx, prec, dagger, a, st);
  auto go = [&](auto tag_s) -> int {
    typedef decltype(tag_s) S;
    if (layout == QDWF_RIRI) {
      return dagger ? run_hop<S, QDWF_RIRI, true>(ctx, prec, a, st, sh)
                    : run_hop<S, QDWF_RIRI, false>(ctx, prec, a, st, sh);
    }
    return dagger ? run_hop<S, QDWF_RRII, true>(ctx, prec, a, st, sh)
                  : run_hop<S, QDWF_RRII, false>(ctx, prec, a, st, sh);
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
