// Launches of the g-SpMM kernels (spmm_kernels.h).
#include "spmm_kernels.h"

namespace gnnk {

bool fast_vec(int dtype, int vec) { return dtype == 0 ? vec == 4 : (vec == 4 || vec == 8); }

namespace {

template <typename T, int V>
void launch_dw_t(const EngineArgs& a, int spec, int gc, dim3 grid, dim3 block, hipStream_t s) {
    if constexpr ((sizeof(T) == 4 && V == 4) || (sizeof(T) == 2 && (V == 4 || V == 8))) {
        // the edge gradient's lane runs (a.red2) as a compile-time constant
        // when they are 2-32 lanes long (the host fuses only runs that fit
        // the lane group), else read at run time
        auto launch = [&](auto cg, auto rg) {
            constexpr int C = decltype(cg)::value;
            constexpr int R = decltype(rg)::value;
            if (spec == SP_UE_H)
                hipLaunchKernelGGL((spmm_sum_kernel<T, V, 1, EXT_NONE, SpUEH<C, false>, R>), grid, block, 0, s, a);
            else
                hipLaunchKernelGGL((spmm_sum_kernel<T, V, 1, EXT_NONE, SpUER<C, false>, R>), grid, block, 0, s, a);
        };
        auto go = [&](auto cg) {
            constexpr int L = 64 / decltype(cg)::value;
            switch (a.red2) {
                case 2: if constexpr (L >= 2) { launch(cg, std::integral_constant<int, 2>{}); return; } break;
                case 4: if constexpr (L >= 4) { launch(cg, std::integral_constant<int, 4>{}); return; } break;
                case 8: if constexpr (L >= 8) { launch(cg, std::integral_constant<int, 8>{}); return; } break;
                case 16: if constexpr (L >= 16) { launch(cg, std::integral_constant<int, 16>{}); return; } break;
                case 32: if constexpr (L >= 32) { launch(cg, std::integral_constant<int, 32>{}); return; } break;
                default: break;
            }
            launch(cg, std::integral_constant<int, 1>{});
        };
        if (gc == 1) go(std::integral_constant<int, 1>{});
        else if (gc == 2) go(std::integral_constant<int, 2>{});
        else go(std::integral_constant<int, 4>{});
    }
}

}  // namespace

hipError_t launch_spmm_dw(const EngineArgs& a, int dtype, int vec, int spec, int gc, hipStream_t s) {
    if (a.sch.w_total <= 0) return hipSuccess;
    const dim3 grid(blocks_for_waves(a.sch.w_total)), block(WAVE * WPB);
    if (dtype == 0) {
        GNNK_VEC_DISPATCH_F32(vec, launch_dw_t<float, V>(a, spec, gc, grid, block, s))
    } else {
        GNNK_VEC_DISPATCH_BF16(vec, launch_dw_t<bf16_t, V>(a, spec, gc, grid, block, s))
    }
    return hipGetLastError();
}

hipError_t launch_spmm(const EngineArgs& a, int dtype, int vec, bool maxmin, int opk, int spec, int gc,
                       hipStream_t s) {
    if (a.sch.w_total <= 0) return hipSuccess;
    const dim3 grid(blocks_for_waves(a.sch.w_total)), block(WAVE * WPB);
    if (a.geo.ov) return launch_spmm_ov(a, dtype, maxmin, opk, spec, gc, grid, block, s);
    const int ext = ext_of(a.flags);
    if (maxmin) {
        if (dtype == 0) {
            GNNK_VEC_DISPATCH_F32(vec, launch_cmp_ov<float, V, false>(a, opk, spec, gc, grid, block, s))
        } else {
            GNNK_VEC_DISPATCH_BF16(vec, launch_cmp_ov<bf16_t, V, false>(a, opk, spec, gc, grid, block, s))
        }
    } else {
        if (dtype == 0) {
            GNNK_VEC_DISPATCH_F32(vec, launch_sum_ov<float, V, false>(a, opk, ext, spec, gc, grid, block, s))
        } else {
            GNNK_VEC_DISPATCH_BF16(vec, launch_sum_ov<bf16_t, V, false>(a, opk, ext, spec, gc, grid, block, s))
        }
    }
    return hipGetLastError();
}

hipError_t launch_spmm_combine(const EngineArgs& a, int dtype, int vec, bool maxmin, hipStream_t s) {
    if (a.sch.n_hub <= 0) return hipSuccess;
    const int64_t waves = (a.sch.n_hub + a.geo.G - 1) / a.geo.G;
    const dim3 grid(blocks_for_waves(waves)), block(WAVE * WPB);
    if (a.geo.ov) return launch_spmm_combine_ov(a, dtype, grid, block, s);  // (sums)
    if (dtype == 0) {
        GNNK_VEC_DISPATCH_F32(vec, launch_combine_t<float, V>(a, maxmin, grid, block, s))
    } else {
        GNNK_VEC_DISPATCH_BF16(vec, launch_combine_t<bf16_t, V>(a, maxmin, grid, block, s))
    }
    return hipGetLastError();
}

}  // namespace gnnk
