// Launch of the column pass of one transfer-function type over all sizes and layouts, for
// complex64 and for 16-bit storage; each type is instantiated in a file of its own (they
// build side by side).
#pragma once
#include "column.hpp"

namespace cwo {

// On the tiled plane a padded column of 8192 runs by default as two transforms of 4096, shorter
// ones as one transform per column; two columns per block in both.
// ALT launchers (single planes, where the autotuner may pick the column form) also build the
// other form at 4096 and 8192: col_form 1 full length, 2 split.
template <class HF, class ST, bool ALT = false>
hipError_t launch_col_t(void* buf, int ny, int my, int mx, int batch, size_t plane,
                               const HF& hf, float hscale, const float2* tw, hipStream_t s,
                               int layout = 0, int col_form = 0) {
    const bool half = (my == 2 * ny);
    using SE = typename ST::E;
    if (layout == 1 && (!half || mx % kTileW != 0)) return hipErrorInvalidValue;
    CWO_DISPATCH_M(my, {
        using C = ColCfg<MM>;
        const int items = (mx + C::COLS - 1) / C::COLS * batch;
        if (half && layout == 1) {
            constexpr bool CAN_SPLIT = MM == 8192 || (ALT && MM == 4096);
            constexpr bool CAN_FULL = MM != 8192 || ALT;
            const bool split = MM == 8192 ? col_form != 1 : col_form == 2;
            if (split) {
                if constexpr (CAN_SPLIT)
                    launch_kernel((k_col_split<MM / 2, HF, ST, LayTile<typename ST::E>>), dim3(mx / 2 * batch),
                                       dim3(MM / 16), 0, s, (SE*)buf, ny, mx, batch, plane, hf,
                                       hscale, tw, LayTile<typename ST::E>{ny});
                else
                    return hipErrorInvalidValue;
            } else {
                if constexpr (CAN_FULL)
                    launch_kernel((k_col<MM, true, HF, ST, LayTile<typename ST::E>>),
                                       dim3(items),
                                       dim3(C::THREADS), 0, s, (SE*)buf, ny, mx, batch, plane, hf,
                                       hscale, tw, LayTile<typename ST::E>{ny});
                else
                    return hipErrorInvalidValue;
            }
        } else if (half) {
            launch_kernel((k_col<MM, true, HF, ST, LayRow>),
                               dim3(items),
                               dim3(C::THREADS), 0, s, (SE*)buf, ny, mx, batch, plane, hf, hscale, tw, LayRow{mx});
        } else if constexpr (std::is_same_v<ST, StF32>) {
            launch_kernel((k_col<MM, false, HF, ST, LayRow>), dim3(items), dim3(C::THREADS),
                               0, s, (SE*)buf, ny, mx, batch, plane, hf, hscale, tw, LayRow{mx});
        } else {
            return hipErrorInvalidValue;
        }
    });
    return hipGetLastError();
}

template <class HF>
hipError_t launch_col_f32(void* buf, int ny, int my, int mx, int batch, size_t plane, const HF& hf,
                          const Storage& st, const float2* tw, hipStream_t s) {
    return launch_col_t<HF, StF32, true>(buf, ny, my, mx, batch, plane, hf, st.col_scale, tw, s,
                                         st.layout, st.col_form);
}

template <class HF>
hipError_t launch_col_16(void* buf, int ny, int my, int mx, int batch, size_t plane, const HF& hf,
                         const Storage& st, const float2* tw, hipStream_t s) {
    if (st.prec == 1)
        return launch_col_t<HF, StF16, true>(buf, ny, my, mx, batch, plane, hf, st.col_scale, tw, s,
                                             st.layout, st.col_form);
    if (st.prec == 2)
        return launch_col_t<HF, StBF16, true>(buf, ny, my, mx, batch, plane, hf, st.col_scale, tw, s,
                                              st.layout, st.col_form);
    return hipErrorInvalidValue;
}

}  // namespace cwo
