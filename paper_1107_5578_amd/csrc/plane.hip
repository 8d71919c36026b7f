// HIP kernels of the diffraction hot path (gfx950).
//
// One propagation of an Ny x Nx complex64 field through the 2Ny x 2Nx padded
// convolution of the paper's convolution-form diffractions (Sec. 2.1.6) is
// three kernels on a [Ny][Mx] complex64 scratch plane:
//
//   row_fwd : for each of the Ny field rows, load Nx values (the Mx - Nx pad
//             values are implicit zeros), forward FFT of length Mx, store the
//             spectrum row. Rows Ny..My-1 of the padded grid are all zero and
//             are never materialised.
//   col     : for each of the Mx columns, load its Ny non-zero rows, forward
//             FFT of length My, multiply by the transfer function of the bin
//             (generated in the kernel), inverse FFT of length My, store the
//             first Ny rows back in place (the crop along y).
//   row_inv : for each of the Ny rows, inverse FFT of length Mx, keep the
//             first Nx values, scale by 1/(Mx*My) and store the output.
//
// Transfer functions (the multiply step of Eqs. ang3 and fre_conv_fft):
//   ASM     : H = exp(i*z*k*sqrt(1 - s)), s = (lambda fx)^2 + (lambda fy)^2,
//             H = 0 for s > 1; the phase in revolutions t = (z/lambda)sqrt(1-s)
//             and its reduction t - rint(t) are FP64, the sine/cosine FP32.
//   Fresnel : H = C * Hx[p] * Hy[q]; the FFT of the sampled impulse response
//             h_F factorises into two 1-D transforms of chirps, computed here
//             by FP64 FFTs.

#include "rowsplit.hpp"

namespace cwo {

// ---- row forward: zero-pad + FFT --------------------------------------------

template <int M, bool HALF, class ST, class IN>
__global__ __launch_bounds__(RowCfg<M>::THREADS) void k_row_fwd(IN ins,
                                                                  typename ST::E* __restrict__ out,
                                                                  int nx, int ny, size_t out_plane,
                                                                  RowScale sc,
                                                                  const float2* __restrict__ tw) {
    using C = RowCfg<M>;
    constexpr int E = C::E, T = C::T;
    const float f = sc.dyn ? sc.in * *sc.dyn : sc.in;
    __shared__ float2 lds[C::RPB * lds_elems<M>()];
    const int tid = threadIdx.x;
    const int sub = tid / T, j = tid % T;
    const int row = blockIdx.x * C::RPB + sub;
    const bool valid = row < ny;
    const float2* src = ins(blockIdx.y) + (size_t)(valid ? row : 0) * nx;
    TwCache<M, fused_of(ST::kFused, M)> twc;
    twc.load(j, tw);
    float2 v[E];
#pragma unroll
    for (int r = 0; r < E; ++r) {
        const int x = j + r * T;
        if constexpr (HALF) {
            // M == 2*nx: exactly the first E/2 registers hold field values
            v[r] = (r < E / 2 && valid) ? ins.value(src[x], row, x) : make_float2(0.f, 0.f);
        } else {
            v[r] = (valid && x < nx) ? ins.value(src[x], row, x) : make_float2(0.f, 0.f);
        }
    }
    if (f != 1.0f) {
#pragma unroll
        for (int r = 0; r < E; ++r) v[r] = make_float2(v[r].x * f, v[r].y * f);
    }
    if constexpr (HALF) fft<M, FWD, 1, true>(v, lds + sub * lds_elems<M>(), j, 0, twc);
    else fft<M, FWD>(v, lds + sub * lds_elems<M>(), j, 0, twc);
    if (valid) {
        typename ST::E* dst = out + blockIdx.y * out_plane + (size_t)row * M;
#pragma unroll
        for (int r = 0; r < E; ++r) dst[j + r * T] = ST::enc(v[r]);
    }
}

// Persistent form: a grid of resident blocks walks the rows (block b takes row groups
// b, b + G, ...) and issues the next group's loads before transforming the current one.
template <int M, bool HALF, class ST, class IN>
__global__ __launch_bounds__(RowCfg<M>::THREADS) void k_row_fwd_pf(IN ins,
                                                                     typename ST::E* __restrict__ out,
                                                                     int nx, int ny, int batch,
                                                                     size_t out_plane, RowScale sc,
                                                                     const float2* __restrict__ tw) {
    using C = RowCfg<M>;
    constexpr int E = C::E, T = C::T;
    constexpr int NL = HALF ? E / 2 : E;
    __shared__ float2 lds[C::RPB * lds_elems<M>()];
    const int tid = threadIdx.x;
    const int sub = tid / T, j = tid % T;
    const float f = sc.dyn ? sc.in * *sc.dyn : sc.in;
    const int rows = ny * batch;
    const int groups = (rows + C::RPB - 1) / C::RPB;
    TwCache<M, fused_of(ST::kFused, M)> twc;
    twc.load(j, tw);
    auto load = [&](int g, float2 (&d)[NL]) {
        const int w = g * C::RPB + sub;
        const bool ok = w < rows;
        const int pl = ok ? w / ny : 0, row = ok ? w - pl * ny : 0;
        const float2* src = ins(pl) + (size_t)row * nx;
#pragma unroll
        for (int r = 0; r < NL; ++r) {
            const int x = j + r * T;
            d[r] = (ok && (HALF || x < nx)) ? ins.value(src[x], row, x) : make_float2(0.f, 0.f);
        }
    };
    float2 cur[NL], nxt[NL];
    int g = blockIdx.x;
    if (g < groups) load(g, cur);
    for (; g < groups; g += gridDim.x) {
        if (g + (int)gridDim.x < groups) load(g + gridDim.x, nxt);
        float2 v[E];
#pragma unroll
        for (int r = 0; r < E; ++r)
            v[r] = r < NL ? make_float2(cur[r].x * f, cur[r].y * f) : make_float2(0.f, 0.f);
        if constexpr (HALF) fft<M, FWD, 1, true>(v, lds + sub * lds_elems<M>(), j, 0, twc);
        else fft<M, FWD>(v, lds + sub * lds_elems<M>(), j, 0, twc);
        const int w = g * C::RPB + sub;
        if (w < rows) {
            const int pl = w / ny, row = w - pl * ny;
            typename ST::E* dst = out + pl * out_plane + (size_t)row * M;
#pragma unroll
            for (int r = 0; r < E; ++r) dst[j + r * T] = ST::enc(v[r]);
        }
#pragma unroll
        for (int r = 0; r < NL; ++r) cur[r] = nxt[r];
    }
}

// ---- row inverse: IFFT + crop + normalisation ---------------------------------

template <int M, bool HALF, class OUT, class ST>
__global__ __launch_bounds__(RowCfg<M>::THREADS) void k_row_inv(
    const typename ST::E* __restrict__ in, OUT outs, int nx, int ny, size_t in_plane, float scale,
    const float* __restrict__ dyn_inv, const float2* __restrict__ tw) {
    using C = RowCfg<M>;
    constexpr int E = C::E, T = C::T;
    if (dyn_inv) scale *= *dyn_inv;
    __shared__ float2 lds[C::RPB * lds_elems<M>()];
    const int tid = threadIdx.x;
    const int sub = tid / T, j = tid % T;
    const int row = blockIdx.x * C::RPB + sub;
    const bool valid = row < ny;
    const typename ST::E* src = in + blockIdx.y * in_plane + (size_t)(valid ? row : 0) * M;
    TwCache<M, fused_of(ST::kFused, M)> twc;
    twc.load(j, tw);
    float2 v[E];
#pragma unroll
    for (int r = 0; r < E; ++r) v[r] = valid ? ST::dec(src[j + r * T]) : make_float2(0.f, 0.f);
    fft<M, INV>(v, lds + sub * lds_elems<M>(), j, 0, twc);
    if (valid) {
        const size_t base = (size_t)row * nx;
        put_row<HALF ? E / 2 : E>(
            outs, blockIdx.y, base + j, T, [&](int r) { return make_float2(v[r].x * scale, v[r].y * scale); },
            [&](int r) { return HALF || j + r * T < nx; });
    }
}

// Persistent form of the row inverse (see k_row_fwd_pf).
template <int M, bool HALF, class OUT, class ST>
__global__ __launch_bounds__(RowCfg<M>::THREADS) void k_row_inv_pf(
    const typename ST::E* __restrict__ in, OUT outs, int nx, int ny, int batch, size_t in_plane,
    float scale, const float* __restrict__ dyn_inv, const float2* __restrict__ tw) {
    using C = RowCfg<M>;
    constexpr int E = C::E, T = C::T;
    __shared__ float2 lds[C::RPB * lds_elems<M>()];
    const int tid = threadIdx.x;
    const int sub = tid / T, j = tid % T;
    if (dyn_inv) scale *= *dyn_inv;
    const int rows = ny * batch;
    const int groups = (rows + C::RPB - 1) / C::RPB;
    TwCache<M, fused_of(ST::kFused, M)> twc;
    twc.load(j, tw);
    using SE = typename ST::E;
    auto load = [&](int g, SE (&d)[E]) {
        const int w = g * C::RPB + sub;
        const bool ok = w < rows;
        const int pl = ok ? w / ny : 0, row = ok ? w - pl * ny : 0;
        const SE* src = in + pl * in_plane + (size_t)row * M;
#pragma unroll
        for (int r = 0; r < E; ++r) d[r] = src[j + r * T];
    };
    SE cur[E], nxt[E];
    int g = blockIdx.x;
    if (g < groups) load(g, cur);
    for (; g < groups; g += gridDim.x) {
        if (g + (int)gridDim.x < groups) load(g + gridDim.x, nxt);
        float2 v[E];
#pragma unroll
        for (int r = 0; r < E; ++r) v[r] = ST::dec(cur[r]);
        fft<M, INV>(v, lds + sub * lds_elems<M>(), j, 0, twc);
        const int w = g * C::RPB + sub;
        if (w < rows) {
            const int pl = w / ny, row = w - pl * ny;
            const size_t base = (size_t)row * nx;
            put_row<HALF ? E / 2 : E>(
                outs, pl, base + j, T, [&](int r) { return make_float2(v[r].x * scale, v[r].y * scale); },
                [&](int r) { return HALF || j + r * T < nx; });
        }
#pragma unroll
        for (int r = 0; r < E; ++r) cur[r] = nxt[r];
    }
}

// ---- row passes on the tiled plane ----------------------------------------------

// Row forward into the tiled plane (padded rows, Mx = 2Nx): ROWS consecutive rows of the
// batch per block, the blocks of one XCD taking a contiguous range of row groups (so the
// rows that share a tile line are written through one L2). The lanes of a wavefront store
// ROWS*kTileW contiguous elements of each tile straight from the transform's registers.
template <int M, class ST, class IN>
__global__ __launch_bounds__(TileRowCfg<M>::THREADS) __attribute__((amdgpu_waves_per_eu(4))) void k_row_fwd_tile(
    IN ins, typename ST::E* __restrict__ out, int nx, int ny, size_t out_plane, RowScale sc,
    const float2* __restrict__ tw) {
    using C = TileRowCfg<M>;
    constexpr int E = kE, T = C::T, NL = E / 2;
    __shared__ float2 lds[C::LDS];
    const int c = threadIdx.x % C::ROWS, j = threadIdx.x / C::ROWS;
    const int w0 = xcd_remap(blockIdx.x, gridDim.x) * C::ROWS, pl = w0 / ny, y0 = w0 - pl * ny;
    const float2* src = ins(pl) + (size_t)y0 * nx;
    const unsigned at = (unsigned)c * nx + j;
    float2 v[E];
#pragma unroll
    for (int r = 0; r < NL; ++r) v[r] = (src + r * T)[at];
    const float f = sc.dyn ? sc.in * *sc.dyn : sc.in;
    TwCache<M, fused_of(ST::kFused, M)> twc;
    twc.load(j, tw);
#pragma unroll
    for (int r = 0; r < NL; ++r) {
        v[r] = ins.value(v[r], y0 + c, j + r * T);
        v[r] = make_float2(v[r].x * f, v[r].y * f);
    }
    fft<M, FWD, C::ROWS, true>(v, lds, j, c, twc);
    const LayTile<typename ST::E> lay{ny};
    typename ST::E* dst = out + pl * out_plane;
    const unsigned to = lay.tile_lane(y0, j / kTileW, T / kTileW) + c * kTileW + j % kTileW;
#pragma unroll
    for (int r = 0; r < E; ++r)
        (dst + lay.tile_step(y0, r * (T / kTileW), T / kTileW))[to] = ST::enc(v[r]);
}

// Row inverse from the tiled plane: the mirror of k_row_fwd_tile; the rows are cropped to the
// first Nx values and scaled.
template <int M, class OUT, class ST>
__global__ __launch_bounds__(TileRowCfg<M>::THREADS) __attribute__((amdgpu_waves_per_eu(4))) void k_row_inv_tile(
    const typename ST::E* __restrict__ in, OUT outs, int nx, int ny, size_t in_plane, float scale,
    const float* __restrict__ dyn_inv, const float2* __restrict__ tw) {
    using C = TileRowCfg<M>;
    constexpr int E = kE, T = C::T;
    __shared__ float2 lds[C::LDS];
    const int c = threadIdx.x % C::ROWS, j = threadIdx.x / C::ROWS;
    if (dyn_inv) scale *= *dyn_inv;
    const int w0 = xcd_remap(blockIdx.x, gridDim.x) * C::ROWS, pl = w0 / ny, y0 = w0 - pl * ny;
    const LayTile<typename ST::E> lay{ny};
    const typename ST::E* src = in + pl * in_plane;
    const unsigned from = lay.tile_lane(y0, j / kTileW, T / kTileW) + c * kTileW + j % kTileW;
    float2 v[E];
#pragma unroll
    for (int r = 0; r < E; ++r)
        v[r] = ST::dec((src + lay.tile_step(y0, r * (T / kTileW), T / kTileW))[from]);
    TwCache<M, fused_of(ST::kFused, M)> twc;
    twc.load(j, tw);
    fft<M, INV, C::ROWS>(v, lds, j, c, twc);
    const size_t base = (size_t)(y0 + c) * nx + j;
    put_row<E / 2>(outs, pl, base, T, [&](int r) { return make_float2(v[r].x * scale, v[r].y * scale); });
}

// ---- tables -------------------------------------------------------------------

// The table of length m (see tw_entries), n values; each evaluated in FP64 and rounded once
// to FP32.
__device__ __forceinline__ float2 unit_root(double num, double den) {
    double s, c;
    sincospi(2.0 * num / den, &s, &c);
    return make_float2((float)c, (float)(-s));
}
__global__ void k_twiddles(float2* tw, int m, int n) {
    int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    float2* const dst = tw + i;
    if (i < m) {
        *dst = unit_root(i, m);
        return;
    }
    // which part (8 or 16 factors, length m or m/2), pass and factor entry i belongs to
    i -= m;
    int per = 8, len = m;
    while (i >= per * tw_pass_k(len)) {
        i -= per * tw_pass_k(len);
        if (len != m) per = 16;
        len = len == m ? m / 2 : m;
    }
    const int bits = ilog2c(len);
    int ns = 1 << ((bits % 4) == 0 ? 4 : bits % 4);
    while (i >= per * ns) {
        i -= per * ns;
        ns <<= 4;
    }
    const int q = i / (2 * ns), k = (i % (2 * ns)) / 2, f = 2 * q + (i & 1);
    // factor f of k: w^a W_16^b with w = exp(-2 pi i k/(16 ns))
    int a = f, b = 0;
    if (per == 8) {
        a = f == 0 ? 8 : f == 1 ? 4 : f < 4 ? 2 : 1;
        b = f == 3 ? 2 : f == 5 ? 2 : f == 6 ? 1 : f == 7 ? 3 : 0;
    }
    if (per == 16) {
        *dst = unit_root((double)(a * k + b * ns), 16.0 * ns);
        return;
    }
    // scale and ratio of exp(-i t): the ratio tan t (cot t from pi/4 on, factors 3, 5 and 7) is
    // rounded first, the scale such that scale and scale * ratio are nearest to cos t and sin t.
    // Only w^8 reaches t = pi/2, at k = ns/2: a scale of 2^-28 puts its factor 2^-28 off -i and
    // leaves room for values up to 2^99.
    const bool cot = f == 3 || f == 5 || f == 7;
    double sn, cs;
    sincospi(2.0 * (double)(a * k + b * ns) / (16.0 * ns), &sn, &cs);
    const double u = cot ? sn : fabs(cs) < 0x1p-28 ? 0x1p-28 : cs, v = cot ? cs : sn;
    const float ratio = (float)(v / u);
    *dst = make_float2((float)((u + v * ratio) / (1.0 + (double)ratio * ratio)), ratio);
}

// ---- host launchers ------------------------------------------------------------

hipError_t launch_twiddles(float2* tw, int m, int n, hipStream_t s) {
    launch_kernel(k_twiddles, dim3((n + 255) / 256), dim3(256), 0, s, tw, m, n);
    return hipGetLastError();
}

template <class ST, class IN>
static hipError_t launch_row_fwd_t(const IN& ins, void* out, int nx, int ny, int mx, int batch,
                                   size_t out_plane, RowScale sc, const float2* tw,
                                   hipStream_t s, int form = 0, int layout = 0) {
    const bool half = (mx == 2 * nx);
    using SE = typename ST::E;
    if (layout == 1) {
        if (!half) return hipErrorInvalidValue;
        CWO_DISPATCH_M(mx, {
            if constexpr (MM == 8192) {
                auto k = k_row_fwd_tsplit<MM / 2, ST, IN>;
                launch_kernel(k, dim3(ny * batch / kSplitRows), dim3(MM / 32 * kSplitRows), 0, s, ins, (SE*)out, nx, ny,
                                   out_plane, sc, tw);
            } else if constexpr (MM >= 512) {
                using C = TileRowCfg<MM>;
                launch_kernel((k_row_fwd_tile<MM, ST, IN>), dim3(ny * batch / C::ROWS),
                                   dim3(C::THREADS), 0, s, ins, (SE*)out, nx, ny, out_plane, sc, tw);
            } else {
                return hipErrorInvalidValue;
            }
        });
        return hipGetLastError();
    }
    // persistent form with prefetch where rows are long enough to fill whole blocks
    // (form 2 asks for one row group per block)
    if (half && mx >= 1024 && form != 2) {
        CWO_DISPATCH_M(mx, {
            if constexpr (MM >= 1024) {
                using C = RowCfg<MM>;
                const int groups = (ny * batch + C::RPB - 1) / C::RPB;
                auto k = k_row_fwd_pf<MM, true, ST, IN>;
                launch_kernel(k, dim3(resident_blocks(k, C::THREADS, groups)), dim3(C::THREADS),
                                   0, s, ins, (SE*)out, nx, ny, batch, out_plane, sc, tw);
            }
        });
        return hipGetLastError();
    }
    CWO_DISPATCH_M(mx, {
        using C = RowCfg<MM>;
        dim3 grid((ny + C::RPB - 1) / C::RPB, batch);
        if (half)
            launch_kernel((k_row_fwd<MM, true, ST, IN>), grid, dim3(C::THREADS), 0, s, ins,
                               (SE*)out, nx, ny, out_plane, sc, tw);
        else if constexpr (std::is_same_v<ST, StF32>)
            launch_kernel((k_row_fwd<MM, false, ST, IN>), grid, dim3(C::THREADS), 0, s, ins,
                               (SE*)out, nx, ny, out_plane, sc, tw);
        else
            return hipErrorInvalidValue;
    });
    return hipGetLastError();
}

hipError_t launch_row_fwd(const float2* in, void* out, int nx, int ny, int mx, int batch,
                          size_t in_plane, size_t out_plane, const Storage& st, const float2* tw,
                          hipStream_t s) {
    const RowScale sc{st.in_scale, st.dyn_scale};
    switch (st.prec) {
        case 0: return launch_row_fwd_t<StF32>(InStrided{in, in_plane}, out, nx, ny, mx, batch, out_plane, sc, tw, s, st.row_form, st.layout);
        case 1: return launch_row_fwd_t<StF16>(InStrided{in, in_plane}, out, nx, ny, mx, batch, out_plane, sc, tw, s, st.row_form, st.layout);
        case 2: return launch_row_fwd_t<StBF16>(InStrided{in, in_plane}, out, nx, ny, mx, batch, out_plane, sc, tw, s, st.row_form, st.layout);
    }
    return hipErrorInvalidValue;
}

hipError_t launch_row_fwd_tab(const InTable& ins, float2* out, int nx, int ny, int mx, int batch,
                              size_t out_plane, const float2* tw, hipStream_t s, int layout) {
    return launch_row_fwd_t<StF32>(ins, out, nx, ny, mx, batch, out_plane,
                                   RowScale{1.0f, nullptr}, tw, s, 0, layout);
}

// Whether the row inverse stores its result past the caches: where a launch's scratch planes
// are more than half of the 256 MiB of the last-level cache, the results would push out the
// scratch that is still to be read. Measured, three passes without and with: one field of
// 4096^2 400 and 366 us (row inverse 105 and 82), 16 fields of 1024^2 382 and 331, 3 of 2048^2
// 246 and 241. With 128 MiB and below a following pass over the result finds it in the cache:
// 8 fields of 1024^2, each result propagated again, 177 and 182; one of 4096^2 in 16-bit
// storage 343 and 350; one of 2048^2 88 and 92.
template <class ST>
static bool past_caches(int ny, int mx, int batch) {
    return (size_t)ny * batch * mx * sizeof(typename ST::E) > (size_t)128 << 20;
}

template <class OUT, class ST>
static hipError_t launch_row_inv_t(const void* in, OUT outs, int nx, int ny, int mx,
                                   int batch, size_t in_plane, float scale, const float* dyn_inv,
                                   const float2* tw, hipStream_t s, int form = 0,
                                   int layout = 0) {
    const bool half = (mx == 2 * nx);
    using SE = typename ST::E;
    outs.nt = past_caches<ST>(ny, mx, batch);
    if (layout == 1) {
        if (!half) return hipErrorInvalidValue;
        CWO_DISPATCH_M(mx, {
            if constexpr (MM == 8192) {
                auto k = k_row_inv_tsplit<MM / 2, OUT, ST>;
                launch_kernel(k, dim3(ny * batch / kSplitRows), dim3(MM / 32 * kSplitRows), 0, s, (const SE*)in, outs, nx, ny,
                                   in_plane, scale, dyn_inv, tw);
            } else if constexpr (MM >= 512) {
                using C = TileRowCfg<MM>;
                launch_kernel((k_row_inv_tile<MM, OUT, ST>), dim3(ny * batch / C::ROWS),
                                   dim3(C::THREADS), 0, s, (const SE*)in, outs, nx, ny, in_plane,
                                   scale, dyn_inv, tw);
            } else {
                return hipErrorInvalidValue;
            }
        });
        return hipGetLastError();
    }
    if (half && mx >= 1024 && form != 2) {
        CWO_DISPATCH_M(mx, {
            if constexpr (MM >= 1024) {
                using C = RowCfg<MM>;
                const int groups = (ny * batch + C::RPB - 1) / C::RPB;
                auto k = k_row_inv_pf<MM, true, OUT, ST>;
                launch_kernel(k, dim3(resident_blocks(k, C::THREADS, groups)), dim3(C::THREADS),
                                   0, s, (const SE*)in, outs, nx, ny, batch, in_plane, scale,
                                   dyn_inv, tw);
            }
        });
        return hipGetLastError();
    }
    CWO_DISPATCH_M(mx, {
        using C = RowCfg<MM>;
        dim3 grid((ny + C::RPB - 1) / C::RPB, batch);
        if (half)
            launch_kernel((k_row_inv<MM, true, OUT, ST>), grid, dim3(C::THREADS), 0, s,
                               (const SE*)in, outs, nx, ny, in_plane, scale, dyn_inv, tw);
        else if constexpr (std::is_same_v<ST, StF32>)
            launch_kernel((k_row_inv<MM, false, OUT, ST>), grid, dim3(C::THREADS), 0, s,
                               (const SE*)in, outs, nx, ny, in_plane, scale, dyn_inv, tw);
        else
            return hipErrorInvalidValue;
    });
    return hipGetLastError();
}

template <class OUT>
static hipError_t launch_row_inv_impl(const float2* in, const OUT& outs, int nx, int ny, int mx,
                                      int batch, size_t in_plane, float scale, const float2* tw,
                                      hipStream_t s, int layout = 0) {
    return launch_row_inv_t<OUT, StF32>(in, outs, nx, ny, mx, batch, in_plane, scale, nullptr, tw,
                                        s, 0, layout);
}

hipError_t launch_row_inv_tab(const float2* in, const OutTable& outs, int nx, int ny, int mx,
                              int batch, size_t in_plane, float scale, const float2* tw,
                              hipStream_t s, int layout) {
    return launch_row_inv_impl(in, outs, nx, ny, mx, batch, in_plane, scale, tw, s, layout);
}

hipError_t launch_row_inv_intensity(const void* in, float* out, int nx, int ny, int mx,
                                    const Storage& st, const float2* tw, hipStream_t s) {
    const OutIntensity o{out, 0};
    switch (st.prec) {
        case 0:
            return launch_row_inv_t<OutIntensity, StF32>(in, o, nx, ny, mx, 1, 0, st.out_scale,
                                                         st.dyn_inv, tw, s, st.row_form, st.layout);
        case 1:
            return launch_row_inv_t<OutIntensity, StF16>(in, o, nx, ny, mx, 1, 0, st.out_scale,
                                                         st.dyn_inv, tw, s, st.row_form, st.layout);
        case 2:
            return launch_row_inv_t<OutIntensity, StBF16>(in, o, nx, ny, mx, 1, 0, st.out_scale,
                                                          st.dyn_inv, tw, s, st.row_form, st.layout);
    }
    return hipErrorInvalidValue;
}

hipError_t launch_row_inv(const void* in, float2* out, int nx, int ny, int mx, int batch,
                          size_t in_plane, size_t out_plane, const Storage& st, const float2* tw,
                          hipStream_t s) {
    const OutStrided o{out, out_plane};
    switch (st.prec) {
        case 0:
            return launch_row_inv_t<OutStrided, StF32>(in, o, nx, ny, mx, batch, in_plane,
                                                       st.out_scale, st.dyn_inv, tw, s,
                                                       st.row_form, st.layout);
        case 1:
            return launch_row_inv_t<OutStrided, StF16>(in, o, nx, ny, mx, batch, in_plane,
                                                       st.out_scale, st.dyn_inv, tw, s,
                                                       st.row_form, st.layout);
        case 2:
            return launch_row_inv_t<OutStrided, StBF16>(in, o, nx, ny, mx, batch, in_plane,
                                                        st.out_scale, st.dyn_inv, tw, s,
                                                        st.row_form, st.layout);
    }
    return hipErrorInvalidValue;
}

// ---- shifted Fresnel: chirps around the row passes -------------------------------

// The field times the source chirp prex[x] prey[y].
struct InChirp {
    const float2* in;
    const float2 *prex, *prey;
    __device__ __forceinline__ const float2* operator()(int) const { return in; }
    __device__ __forceinline__ float2 value(float2 v, int y, int x) const {
        return cmul(v, cmul(prex[x], prey[y]));
    }
};
// The result times the destination chirp postx[x] posty[y] (nx a power of two).
struct OutChirp {
    float2* out;
    const float2 *postx, *posty;
    int nx, lognx;
    bool nt = false;
    template <bool NT>
    __device__ __forceinline__ void put(int, size_t i, float2 v) const {
        store<NT>(out + i, cmul(v, cmul(postx[i & (nx - 1)], posty[i >> lognx])));
    }
};

hipError_t launch_sf_row_fwd(const float2* in, float2* out, int nx, int ny, const float2* tabs,
                             const float2* tw, hipStream_t s, int layout) {
    return launch_row_fwd_t<StF32>(InChirp{in, tabs, tabs + nx}, out, nx, ny, 2 * nx, 1, 0,
                                   RowScale{1.0f, nullptr}, tw, s, 0, layout);
}

hipError_t launch_sf_row_inv(const float2* in, float2* out, int nx, int ny, float scale,
                             const float2* tabs, const float2* tw, hipStream_t s, int layout) {
    const float2* postx = tabs + nx + ny;
    return launch_row_inv_t<OutChirp, StF32>(in, OutChirp{out, postx, postx + nx, nx, ilog2c(nx)},
                                             nx, ny, 2 * nx, 1, 0, scale, nullptr, tw, s, 0, layout);
}

// ---- range of a field for FP16 storage -----------------------------------------

__device__ __forceinline__ float absmax(float2 v) { return fmaxf(fabsf(v.x), fabsf(v.y)); }
__device__ __forceinline__ float absmax(float v) { return fabsf(v); }

// Maximum over a block of 256 threads (thread 0's result).
__device__ __forceinline__ float block_max(float m) {
    __shared__ float red[4];
#pragma unroll
    for (int d = 32; d > 0; d >>= 1) m = fmaxf(m, __shfl_xor(m, d));
    if (threadIdx.x % 64 == 0) red[threadIdx.x / 64] = m;
    __syncthreads();
    return fmaxf(fmaxf(red[0], red[1]), fmaxf(red[2], red[3]));
}

// Per-block maximum of |re|, |im| (of |a| for a real array) over a grid-strided range. Eight
// loads in flight per thread and shuffles in place of a tree in LDS: what is left is the
// two launches. FP16 planes with loads one after another and now: 512^2 22.9 and 21 us, 1024^2
// 35.5 and 33.7 (37.4 and 34.7 on new inputs), 4096^2 361 and 357.
template <class T>
__global__ __launch_bounds__(256) void k_absmax_partial(const T* __restrict__ in, size_t n,
                                                        float* __restrict__ partial) {
    constexpr int U = 8;
    const size_t step = (size_t)gridDim.x * 256;
    size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
    float m = 0.f;
    for (; i + (U - 1) * step < n; i += U * step) {
        T x[U];
#pragma unroll
        for (int k = 0; k < U; ++k) x[k] = in[i + k * step];
#pragma unroll
        for (int k = 0; k < U; ++k) m = fmaxf(m, absmax(x[k]));
    }
    for (; i < n; i += step) m = fmaxf(m, absmax(in[i]));
    m = block_max(m);
    if (threadIdx.x == 0) partial[blockIdx.x] = m;
}

// scale[0] = 2^-e with e = ceil(log2(max)) (so the scaled field is within [-1, 1]),
// scale[1] = 2^e; both 1 when the field is zero or not finite
__global__ __launch_bounds__(256) void k_absmax_final(const float* __restrict__ partial, int np,
                                                      float* __restrict__ scale) {
    float m = 0.f;
    for (int i = threadIdx.x; i < np; i += 256) m = fmaxf(m, partial[i]);
    const float mx = block_max(m);
    if (threadIdx.x == 0) {
        int e = 0;
        if (mx > 0.f && isfinite(mx)) {
            const float f = frexpf(mx, &e);  // mx = f * 2^e, f in [0.5, 1)
            (void)f;
        }
        scale[0] = ldexpf(1.0f, -e);
        scale[1] = ldexpf(1.0f, e);
    }
}

namespace {
template <class T>
hipError_t range_scale_t(const T* in, size_t n, float* work, hipStream_t s) {
    const size_t want = (n + 256 * 16 - 1) / (256 * 16);
    const int nb = want < 1 ? 1 : (want < (size_t)kRangeBlocks ? (int)want : kRangeBlocks);
    launch_kernel((k_absmax_partial<T>), dim3(nb), dim3(256), 0, s, in, n, work + 2);
    launch_kernel(k_absmax_final, dim3(1), dim3(256), 0, s, (const float*)(work + 2), nb, work);
    return hipGetLastError();
}
}  // namespace

hipError_t launch_range_scale(const float2* in, size_t n, float* work, hipStream_t s) {
    return range_scale_t(in, n, work, s);
}

hipError_t launch_range_scale(const float* in, size_t n, float* work, hipStream_t s) {
    return range_scale_t(in, n, work, s);
}

}  // namespace cwo
