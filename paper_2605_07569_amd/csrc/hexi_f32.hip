// The fp32 kernels on the fp32 matrix instruction (units: hexi_f32_units.h) and the dispatch of the fp32 path.
#include "hexi_f32_units.h"
#include "hexi_shapes.h"

namespace {

template <int D, bool SPLIT, bool TWO, int CHAINS> using Cfg = rows16::F32Cfg<D, SPLIT, TWO, SPLIT ? 8 : 4, CHAINS>;

template <int D, bool SPLIT, bool TWO, int CHAINS>
__global__ void __launch_bounds__((64 * Cfg<D, SPLIT, TWO, CHAINS>::NW), TWO ? 4 : 1) fwd_f32_kernel(const FwdArgs a, const int n_q_tiles)
{
    using C = Cfg<D, SPLIT, TWO, CHAINS>;
    __shared__ __attribute__((aligned(1024))) rows16::FwdSmem<C> sm;
    // heads of a q tile side by side, the longest (last) q tiles first
    rows16::fwd_unit<C>(a, blockIdx.x % a.g.nq, n_q_tiles - 1 - blockIdx.x / a.g.nq, sm);
}

// The backward step in one launch: workgroups [0, n_dkdv) are dK / dV units (the longer ones, first), the others dQ units; heads
// side by side, the longest tiles first.  As two launches, each left CUs idle at its end: 2600 keys of 2 kv heads are 324
// workgroups of equal length, two rounds of 256 CUs with the second one a quarter full.  3055 rows x 12011 keys, 6 / 2 heads,
// forward + backward: 3.24 -> 2.77 ms.  Two shared workgroups are to fit a CU: 256 registers, which four chains would exceed by 20.
template <int D, bool SPLIT, bool TWO, int CHAINS>
__global__ void __launch_bounds__((64 * Cfg<D, SPLIT, TWO, CHAINS>::NW), TWO ? 4 : SPLIT ? 1 : 2) bwd_f32_kernel(const BwdArgs a, const unsigned n_dkdv, const int n_q_tiles)
{
    using C = Cfg<D, SPLIT, TWO, CHAINS>;
    __shared__ __attribute__((aligned(1024))) union { rows16::DkdvSmem<C> dkdv; rows16::DqSmem<C> dq; } sm;
    if (blockIdx.x < n_dkdv) {
        const int tile = __builtin_amdgcn_readfirstlane(blockIdx.x / (unsigned)a.g.nkv);
        rows16::dkdv_unit<C>(a, (int)blockIdx.x - tile * a.g.nkv, tile, sm.dkdv, 0, a.g.nq, false);
    } else {
        const unsigned unit = blockIdx.x - n_dkdv;
        const int tile = __builtin_amdgcn_readfirstlane(unit / (unsigned)a.g.nq);
        rows16::dq_unit<C>(a, (int)unit - tile * a.g.nq, n_q_tiles - 1 - tile, sm.dq);
    }
}

// f(configuration).
template <class F> hipError_t with_cfg(const AttnGeom& g, F32Shape shape, F f)
{
    const bool split = shape != F32Shape::SHARED;
    if (g.d == 128 && hexi_f32_chains(g) == 4) { if (split) f(Cfg<128, true, false, 4>{}); else f(Cfg<128, false, false, 4>{}); }
    else if (g.d == 128) { if (split) f(Cfg<128, true, false, 1>{}); else f(Cfg<128, false, false, 1>{}); }
    else if (g.d != 64) return hipErrorInvalidValue;
    else if (shape == F32Shape::SPLIT_TWO) f(Cfg<64, true, true, 1>{});
    else if (split) f(Cfg<64, true, false, 1>{});
    else f(Cfg<64, false, false, 1>{});
    return hipGetLastError();
}

}  // namespace

hipError_t hexi_launch_fwd_f32(const FwdArgs& a, hipStream_t s)
{
    if (const F32x3Fwd plan = hexi_f32x3_fwd(a.g); plan.use) return hexi_launch_fwd_f32x3(a, plan, s);
    return with_cfg(a.g, hexi_f32_fwd_shape(a.g), [&](auto cfg) {
        using C = decltype(cfg);
        const int n_q_tiles = (a.g.lq + C::ROWS - 1) / C::ROWS;
        fwd_f32_kernel<C::D, C::SPLIT, C::TWO, C::CHAINS><<<(unsigned)(n_q_tiles * a.g.nq), 64 * C::NW, 0, s>>>(a, n_q_tiles);
    });
}

hipError_t hexi_launch_bwd_f32(const BwdArgs& a, hipStream_t s)
{
    if (const F32x3Bwd plan = hexi_f32x3_bwd(a.g, a.accumulate != 0, a.want_dq != 0, a.want_dkdv != 0, hexi_dkdv_run_len); plan.use) return hexi_launch_bwd_f32x3(a, plan, s);
    F32Shape kv_shape, q_shape;
    hexi_f32_bwd_shapes(a.g, a.want_dq, a.want_dkdv, &kv_shape, &q_shape);
    auto launch = [&](F32Shape shape, bool dkdv, bool dq) {
        return with_cfg(a.g, shape, [&](auto cfg) {
            using C = decltype(cfg);
            const int n_q_tiles = (a.g.lq + C::ROWS - 1) / C::ROWS;
            const unsigned n_dkdv = dkdv ? (unsigned)((a.g.lc + C::ROWS - 1) / C::ROWS * a.g.nkv) : 0u;
            const unsigned n_dq = dq ? (unsigned)(n_q_tiles * a.g.nq) : 0u;
            bwd_f32_kernel<C::D, C::SPLIT, C::TWO, C::CHAINS><<<n_dkdv + n_dq, 64 * C::NW, 0, s>>>(a, n_dkdv, n_q_tiles);
        });
    };
    if (a.want_dkdv && a.want_dq && kv_shape == q_shape) return launch(kv_shape, true, true);
    hipError_t e = a.want_dkdv ? launch(kv_shape, true, false) : hipSuccess;
    if (e == hipSuccess && a.want_dq) e = launch(q_shape, false, true);
    return e;
}
