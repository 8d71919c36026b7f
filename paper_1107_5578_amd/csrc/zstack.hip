// HIP kernels of the z-stack form (one field, many distances): the forward column
// transform once per column, then per plane the transfer function, the inverse column
// transform and the row inverse.

#include "kernel_common.hpp"

namespace cwo {

// ---- z-stack column pass ------------------------------------------------------
//
// One field, many distances: the forward column transform is done once per column
// and kept in registers; for each plane the spectrum is multiplied by that plane's
// transfer function and inverse transformed into the plane's scratch.

// The z-independent part of each bin is computed once, after the forward column
// transform, and kept across the plane loop; each plane then costs one FP64 multiply
// and a reduction per bin.
//
// Fast form (every bin s <= 0.05): K = 1 - sqrt(1 - s) = s/2 + T(s) from the same
// series as AsmHFast; minus the phase of plane z is zl*K - zl revolutions, reduced to [0, 1)
// in FP64. 16-bit storage and short columns (see fused_of) keep reduce(zl) - reduce(zl*K),
// subtracted in FP32 (more exact there: 2.53e-7 of a plane's norm at 128^2, else 2.55e-7).
// Exact form: Q = sqrt(1 - s) in FP64 (Q < 0 marks an evanescent bin, s > 1, decided with
// the reference's operations); the phase is zl*Q.
struct AsmZFast {
    double lam_dfx, lam_dfy;
    int mx, my;
    __device__ __forceinline__ double bin(int p, int q) const {
        const double x = (double)(p < mx / 2 ? p : p - mx) * lam_dfx;
        const double y = (double)(q < my / 2 ? q : q - my) * lam_dfy;
        const double s = x * x + y * y;
        double poly = 715.0 / 65536.0;
        poly = fma(poly, s, 429.0 / 32768.0);
        poly = fma(poly, s, 33.0 / 2048.0);
        poly = fma(poly, s, 21.0 / 1024.0);
        poly = fma(poly, s, 7.0 / 256.0);
        poly = fma(poly, s, 5.0 / 128.0);
        poly = fma(poly, s, 1.0 / 16.0);
        poly = fma(poly, s, 1.0 / 8.0);
        return fma(s * s, poly, 0.5 * s);
    }
    // zr: rint(zl) - zl
    template <bool FUSED>
    __device__ __forceinline__ float2 at(double k, double zl, double zr) const {
        if constexpr (FUSED) {
            const float r = (float)__builtin_amdgcn_fract(fma(zl, k, zr));
            return make_float2(__builtin_amdgcn_cosf(r), -__builtin_amdgcn_sinf(r));
        } else {
            const double u = zl * k;
            float r = (float)-zr - (float)(u - rint(u));
            r -= rintf(r);
            return make_float2(__builtin_amdgcn_cosf(r), __builtin_amdgcn_sinf(r));
        }
    }
};

struct AsmZExact {
    double dfx, dfy, lam;
    int mx, my;
    __device__ __forceinline__ double bin(int p, int q) const {
#pragma clang fp contract(off)
        const double pp = (double)(p < mx / 2 ? p : p - mx);
        const double qq = (double)(q < my / 2 ? q : q - my);
        const double ax = lam * (pp * dfx);
        const double ay = lam * (qq * dfy);
        const double s = ay * ay + ax * ax;
        return (s <= 1.0) ? sqrt(1.0 - s) : -1.0;
    }
    template <bool>
    __device__ __forceinline__ float2 at(double qv, double zl, double) const {
        if (qv < 0.0) return make_float2(0.f, 0.f);
        const double t = zl * qv;
        const float r = (float)(t - rint(t));
        return make_float2(__builtin_amdgcn_cosf(r), __builtin_amdgcn_sinf(r));
    }
};

template <class ZH>
struct ZSetAsm {
    ZH h;
    double zl[kZChunk];
    int nz;
};

struct ZSetFresnel {
    const float2* h;  // plane k: Hx (with C) at h + k*stride, Hy at h + k*stride + mx
    size_t stride;
    int mx, nz;
};

// The z-stack planes are stored in groups of W adjacent columns: element (y, x) at
// ((x/W)*ny + y)*W + x%W. The column pass writes a group's rows one after another, so its
// lines are whole when they leave the L2 (row-major stores of single columns would leave
// partially written ones), and the row inverse reads W values of each of its rows at a time.
// Row inverse against column-major planes: 64 planes of 1024^2 (W = 2) 420 -> 366 us, of
// 512^2 109 -> 96, 16 of 2048^2 574 -> 430 for 11 us more in the column pass, whose blocks
// there hold one column and share lines with their neighbours (W = 4: 374, but 82 more).
// Spreading the groups over the channels, as the tiled plane does, takes 398 us at 1024^2.
template <int M>
constexpr int z_width() {
    return M >= 4096 ? 2 : ZColCfg<M>::COLS < 4 ? ZColCfg<M>::COLS : 4;
}

// Column pass of one block: COLS columns, the planes [k0, k1) of the launch. factor(k) gives
// the transfer function of plane k as a function of the register index.
template <int M, bool HALF, class ST, class TW, class F>
__device__ __forceinline__ void zcol_planes(const float2 (&v)[kE], typename ST::E* __restrict__ zbuf,
                                            int ny, size_t zplane, int col, bool active, int k0,
                                            int k1, float hscale, float2* lds, int j, int c,
                                            const TW& twc, F&& factor) {
    constexpr int T = ZColCfg<M>::T, W = z_width<M>();
    for (int k = k0; k < k1; ++k) {
        float2 w[kE];
#pragma unroll
        for (int r = 0; r < kE; ++r) w[r] = v[r];
        fft_mul<M, INV, ZColCfg<M>::COLS>(w, factor(k), lds, j, c, twc);
        typename ST::E* dst = zbuf + (size_t)k * zplane + (size_t)(col / W) * ny * W + col % W;
#pragma unroll
        for (int r = 0; r < kE; ++r) {
            if constexpr (!std::is_same_v<ST, StF32>) w[r] = make_float2(w[r].x * hscale, w[r].y * hscale);
            if (active && (HALF ? (r < kE / 2) : (j + r * T < ny)))
                (dst + r * T * W)[(unsigned)j * W] = ST::enc(w[r]);
        }
    }
}

// Forward transform of a block's columns of the shared spectrum.
template <int M, bool HALF, class ST, class TW>
__device__ __forceinline__ void zcol_forward(const typename ST::E* __restrict__ src, int ny, int mx,
                                             int j, int c, bool active, float2 (&v)[kE], float2* lds,
                                             const TW& twc) {
    constexpr int T = ZColCfg<M>::T;
#pragma unroll
    for (int r = 0; r < kE; ++r) {
        const bool ld = active && (HALF ? (r < kE / 2) : (j + r * T < ny));
        v[r] = ld ? ST::dec(src[(size_t)(j + r * T) * mx]) : make_float2(0.f, 0.f);
    }
    fft<M, FWD, ZColCfg<M>::COLS, HALF>(v, lds, j, c, twc);
}

// The z-independent factor of each bin stays in registers beside the forward spectrum and the
// twiddles: 166 VGPRs, three waves per SIMD and no LDS beyond the exchange (parked in LDS it
// held blocks to two waves: 421 us per 64 planes of 1024^2, now 326 to 335, of which 277 are vector
// issue). 16-bit storage holds twice the twiddles: two waves.
template <int M, bool HALF, class ZH, class ST>
__global__ __launch_bounds__(ZColCfg<M>::THREADS) __attribute__((amdgpu_waves_per_eu(ST::kFused ? 3 : 2))) void k_col_z_asm(
    const typename ST::E* __restrict__ spec, typename ST::E* __restrict__ zbuf, int ny, int mx,
    size_t zplane, ZSetAsm<ZH> zs, float hscale, const float2* __restrict__ tw) {
    using C = ZColCfg<M>;
    constexpr int E = kE, T = C::T;
    __shared__ float2 lds[C::LDS];
    const int c = threadIdx.x % C::COLS, j = threadIdx.x / C::COLS;
    int col0 = xcd_remap(blockIdx.x, gridDim.x) * C::COLS + c;
    // (opaque: as a uniform value of a one-column block it made the planes' loop 4 % slower)
    asm volatile("" : "+v"(col0));
    const bool active = col0 < mx;
    const int col = active ? col0 : 0;
    TwCache<M, fused_of(ST::kFused, M)> twc;
    twc.load(j, tw);
    float2 v[E];
    zcol_forward<M, HALF, ST>(spec + col, ny, mx, j, c, active, v, lds, twc);
    double kb[E];
#pragma unroll
    for (int r = 0; r < E; ++r) kb[r] = zs.h.bin(col, j + r * T);
    const int per = (zs.nz + gridDim.y - 1) / gridDim.y, k0 = blockIdx.y * per;
    zcol_planes<M, HALF, ST>(v, zbuf, ny, zplane, col, active, k0, min(zs.nz, k0 + per), hscale,
                             lds, j, c, twc, [&](int k) {
                                 const double zl = zs.zl[k];
                                 const double zr = rint(zl) - zl;
                                 return [&kb, &zs, zl, zr](auto rc) {
                                     return zs.h.template at<fused_of(ST::kFused, M)>(kb[decltype(rc)::value], zl, zr);
                                 };
                             });
}

template <int M, bool HALF, class ST>
__global__ __launch_bounds__(ZColCfg<M>::THREADS) __attribute__((amdgpu_waves_per_eu(ST::kFused ? 3 : 2))) void k_col_z_fresnel(
    const typename ST::E* __restrict__ spec, typename ST::E* __restrict__ zbuf, int ny, int mx,
    size_t zplane, ZSetFresnel zs, float hscale, const float2* __restrict__ tw) {
    using C = ZColCfg<M>;
    constexpr int E = kE, T = C::T;
    __shared__ float2 lds[C::LDS];
    const int c = threadIdx.x % C::COLS, j = threadIdx.x / C::COLS;
    int col0 = xcd_remap(blockIdx.x, gridDim.x) * C::COLS + c;
    // (opaque: as a uniform value of a one-column block it made the planes' loop 4 % slower)
    asm volatile("" : "+v"(col0));
    const bool active = col0 < mx;
    const int col = active ? col0 : 0;
    TwCache<M, fused_of(ST::kFused, M)> twc;
    twc.load(j, tw);
    float2 v[E];
    zcol_forward<M, HALF, ST>(spec + col, ny, mx, j, c, active, v, lds, twc);
    const int per = (zs.nz + gridDim.y - 1) / gridDim.y, k0 = blockIdx.y * per;
    zcol_planes<M, HALF, ST>(v, zbuf, ny, zplane, col, active, k0, min(zs.nz, k0 + per), hscale,
                             lds, j, c, twc, [&](int k) {
                                 const float2* hk = zs.h + (size_t)k * zs.stride;
                                 const float2 hx = hk[col];
                                 const float2* hy = hk + zs.mx + j;
                                 return [hx, hy](auto rc) {
                                     return cmul(hx, (hy + decltype(rc)::value * T)[0]);
                                 };
                             });
}

// Row inverse of z-stack planes (in groups of 2^lw columns, as the z-stack column pass writes
// them): COLS adjacent rows in consecutive lanes, one row per thread; rows are stored to the row-major outputs with the crop and the
// 1/(Mx*My) scale. Tiles of rows are taken in XCD-contiguous ranges, so the blocks that share
// an input cache line share an L2.
template <int M, bool HALF, class OUT, class ST>
__global__ __launch_bounds__(ZRowCfg<M>::THREADS) __attribute__((amdgpu_waves_per_eu(ZRowCfg<M>::WAVES_PER_EU))) void k_row_inv_t(
    const typename ST::E* __restrict__ in, OUT outs, int nx, int ny, int lw, size_t in_plane,
    float scale, const float* __restrict__ dyn_inv, const float2* __restrict__ tw) {
    using C = ZRowCfg<M>;
    constexpr int E = kE, T = C::T;
    using SE = typename ST::E;
    if (dyn_inv) scale *= *dyn_inv;
    __shared__ float2 lds[C::LDS];
    const int c = threadIdx.x % C::COLS, j = threadIdx.x / C::COLS;
    const int ntiles = (ny + C::COLS - 1) / C::COLS;
    const int it = xcd_remap(blockIdx.x, gridDim.x);
    const int pl = it / ntiles, tile = it - pl * ntiles;
    const int y0 = tile * C::COLS + c;
    const bool active = C::COLS <= 16 || y0 < ny;
    const int y = active ? y0 : 0;
    const SE* base = in + pl * in_plane;
    auto place = [&](unsigned x) { return (((x >> lw) * ny + y) << lw) + (x & ((1u << lw) - 1)); };
    const unsigned at = place(j);
    float2 v[E];
#pragma unroll
    for (int r = 0; r < E; ++r) {
        if constexpr (T >= 4) v[r] = ST::dec((base + (size_t)(r * T) * ny)[at]);
        else v[r] = ST::dec(base[place(j + r * T)]);
    }
    TwCache<M, fused_of(ST::kFused, M), !ST::kFused> twc;
    twc.load(j, tw);
    fft<M, INV, C::COLS>(v, lds, j, c, twc);
    if (!active) return;  // after the last exchange: no barrier follows
    const size_t o = (size_t)y * nx + j;
#pragma unroll
    for (int r = 0; r < E; ++r) {
        if (HALF ? (r < E / 2) : (j + r * T < nx))
            outs.template put<false>(pl, o + r * T, make_float2(v[r].x * scale, v[r].y * scale));
    }
}

// ---- host launchers ------------------------------------------------------------

namespace {
// Blocks of the column passes per column tile: the planes of a launch are cut into g groups
// that each repeat the forward transform (about 1.5 planes' time with its loads), g chosen for
// the least number of rounds of resident blocks times the planes' and that time. 64 planes of
// 256^2 have 64 column tiles for 768 places: one group took 151 us, the chosen ones 34.
int z_groups(int tiles, int slots, int nz) {
    int best = 1;
    double least = 0.0;
    for (int g = 1; g <= nz; ++g) {
        const int per = (nz + g - 1) / g;
        if ((long long)per * (g - 1) >= nz) continue;  // the last group would be empty
        const double rounds = ((long long)tiles * g + slots - 1) / slots;
        const double t = rounds * (per + 1.5);
        if (g == 1 || t < 0.97 * least) {
            least = t;
            best = g;
        }
    }
    return best;
}

template <class ST>
hipError_t row_inv_z_t(const void* zbuf, const ZChunk& zc, int nx, int ny, int mx, int my, size_t zplane,
                       float scale, const float* dyn_inv, const float2* tw, hipStream_t s) {
    using SE = typename ST::E;
    OutTable t;
    for (int k = 0; k < kZChunk; ++k) t.out[k] = k < zc.nz ? zc.out[k] : nullptr;
    const bool half = (mx == 2 * nx);
    int lw = 0;
    CWO_DISPATCH_M(my, lw = ilog2c(z_width<MM>()));
    CWO_DISPATCH_M(mx, {
        using C = ZRowCfg<MM>;
        const int items = (ny + C::COLS - 1) / C::COLS * zc.nz;
        if (half)
            launch_kernel((k_row_inv_t<MM, true, OutTable, ST>), dim3(items), dim3(C::THREADS), 0, s,
                               (const SE*)zbuf, t, nx, ny, lw, zplane, scale, dyn_inv, tw);
        else if constexpr (std::is_same_v<ST, StF32>)
            launch_kernel((k_row_inv_t<MM, false, OutTable, ST>), dim3(items),
                               dim3(C::THREADS), 0, s, (const SE*)zbuf, t, nx, ny, lw, zplane,
                               scale, dyn_inv, tw);
        else
            return hipErrorInvalidValue;
    });
    return hipGetLastError();
}

template <class ZH, class ST>
hipError_t col_z_asm_t(const void* spec, void* zbuf, int ny, int my, int mx, size_t zplane,
                       const ZSetAsm<ZH>& zs, float hscale, const float2* tw, hipStream_t s) {
    using SE = typename ST::E;
    const bool half = (my == 2 * ny);
    CWO_DISPATCH_M(my, {
        using C = ZColCfg<MM>;
        const int tiles = (mx + C::COLS - 1) / C::COLS, nz = zs.nz;
        if (half)
            launch_kernel((k_col_z_asm<MM, true, ZH, ST>),
                               dim3(tiles, z_groups(tiles, resident_blocks(k_col_z_asm<MM, true, ZH, ST>, C::THREADS, 1 << 30), nz)),
                               dim3(C::THREADS), 0, s,
                               (const SE*)spec, (SE*)zbuf, ny, mx, zplane, zs, hscale, tw);
        else if constexpr (std::is_same_v<ST, StF32>)
            launch_kernel((k_col_z_asm<MM, false, ZH, ST>),
                               dim3(tiles, z_groups(tiles, resident_blocks(k_col_z_asm<MM, false, ZH, ST>, C::THREADS, 1 << 30), nz)),
                               dim3(C::THREADS), 0, s,
                               (const SE*)spec, (SE*)zbuf, ny, mx, zplane, zs, hscale, tw);
        else
            return hipErrorInvalidValue;
    });
    return hipGetLastError();
}

template <class ST>
hipError_t col_z_fresnel_t(const void* spec, void* zbuf, int ny, int my, int mx, size_t zplane,
                           const ZSetFresnel& zs, float hscale, const float2* tw, hipStream_t s) {
    using SE = typename ST::E;
    const bool half = (my == 2 * ny);
    CWO_DISPATCH_M(my, {
        using C = ZColCfg<MM>;
        const int tiles = (mx + C::COLS - 1) / C::COLS, nz = zs.nz;
        if (half)
            launch_kernel((k_col_z_fresnel<MM, true, ST>),
                               dim3(tiles, z_groups(tiles, resident_blocks(k_col_z_fresnel<MM, true, ST>, C::THREADS, 1 << 30), nz)),
                               dim3(C::THREADS), 0, s,
                               (const SE*)spec, (SE*)zbuf, ny, mx, zplane, zs, hscale, tw);
        else if constexpr (std::is_same_v<ST, StF32>)
            launch_kernel((k_col_z_fresnel<MM, false, ST>),
                               dim3(tiles, z_groups(tiles, resident_blocks(k_col_z_fresnel<MM, false, ST>, C::THREADS, 1 << 30), nz)),
                               dim3(C::THREADS), 0, s,
                               (const SE*)spec, (SE*)zbuf, ny, mx, zplane, zs, hscale, tw);
        else
            return hipErrorInvalidValue;
    });
    return hipGetLastError();
}

template <class ZH>
hipError_t col_z_asm_prec(const void* spec, void* zbuf, int ny, int my, int mx, size_t zplane,
                          const ZSetAsm<ZH>& zs, const Storage& st, const float2* tw,
                          hipStream_t s) {
    switch (st.prec) {
        case 0: return col_z_asm_t<ZH, StF32>(spec, zbuf, ny, my, mx, zplane, zs, st.col_scale, tw, s);
        case 1: return col_z_asm_t<ZH, StF16>(spec, zbuf, ny, my, mx, zplane, zs, st.col_scale, tw, s);
        case 2: return col_z_asm_t<ZH, StBF16>(spec, zbuf, ny, my, mx, zplane, zs, st.col_scale, tw, s);
    }
    return hipErrorInvalidValue;
}
}  // namespace

hipError_t launch_row_inv_z(const void* zbuf, const ZChunk& zc, int nx, int ny, int mx, int my,
                            size_t zplane, const Storage& st, const float2* tw, hipStream_t s) {
    switch (st.prec) {
        case 0: return row_inv_z_t<StF32>(zbuf, zc, nx, ny, mx, my, zplane, st.out_scale, st.dyn_inv, tw, s);
        case 1: return row_inv_z_t<StF16>(zbuf, zc, nx, ny, mx, my, zplane, st.out_scale, st.dyn_inv, tw, s);
        case 2: return row_inv_z_t<StBF16>(zbuf, zc, nx, ny, mx, my, zplane, st.out_scale, st.dyn_inv, tw, s);
    }
    return hipErrorInvalidValue;
}

hipError_t launch_col_z_asm(const void* spec, void* zbuf, int ny, int my, int mx, size_t zplane,
                            const AsmScalars& a, const ZChunk& zc, const Storage& st,
                            const float2* tw, hipStream_t s) {
    const double sx = a.lam * (0.5 * mx) * a.dfx, sy = a.lam * (0.5 * my) * a.dfy;
    if (sx * sx + sy * sy <= kAsmFastMaxS) {
        ZSetAsm<AsmZFast> zs;
        zs.h = AsmZFast{a.lam * a.dfx, a.lam * a.dfy, mx, my};
        for (int k = 0; k < kZChunk; ++k) zs.zl[k] = k < zc.nz ? zc.zl[k] : 0.0;
        zs.nz = zc.nz;
        return col_z_asm_prec(spec, zbuf, ny, my, mx, zplane, zs, st, tw, s);
    }
    ZSetAsm<AsmZExact> zs;
    zs.h = AsmZExact{a.dfx, a.dfy, a.lam, mx, my};
    for (int k = 0; k < kZChunk; ++k) zs.zl[k] = k < zc.nz ? zc.zl[k] : 0.0;
    zs.nz = zc.nz;
    return col_z_asm_prec(spec, zbuf, ny, my, mx, zplane, zs, st, tw, s);
}

hipError_t launch_col_z_fresnel(const void* spec, void* zbuf, int ny, int my, int mx,
                                size_t zplane, const float2* h, int nz, const Storage& st,
                                const float2* tw, hipStream_t s) {
    const ZSetFresnel zs{h, (size_t)(mx + my), mx, nz};
    switch (st.prec) {
        case 0: return col_z_fresnel_t<StF32>(spec, zbuf, ny, my, mx, zplane, zs, st.col_scale, tw, s);
        case 1: return col_z_fresnel_t<StF16>(spec, zbuf, ny, my, mx, zplane, zs, st.col_scale, tw, s);
        case 2: return col_z_fresnel_t<StBF16>(spec, zbuf, ny, my, mx, zplane, zs, st.col_scale, tw, s);
    }
    return hipErrorInvalidValue;
}

}  // namespace cwo
