// HIP kernels of the amplitude-constrained ping-pong iteration (the column pass is the
// plain one).

#include "rowsplit.hpp"

namespace cwo {

// ---- ping-pong iteration row kernel ----------------------------------------------
//
// Row inverse transform, crop, amplitude constraint and re-padded forward transform
// fused, so one propagation of the iteration is a column pass plus this kernel.
// ST is the storage of the padded spectrum. The stored rows carry a power-of-two factor:
// the inverse transform is multiplied by scale * (*dyn_inv) to give the physical field,
// and the constrained field by fwd_scale * (*dyn_fwd) before the forward transform (null
// dyn pointers count as 1), so FP16 storage stays in range.

// Error partials per row for rows of m points (the same for every kernel of that length: the
// buffer holds iterations * ny * this).
constexpr int gs_partials_per_row(int m) { return m / 16 < 64 ? 1 : m / 16 / 64; }

// Error partials of rows of M points, P per row: each thread's double summed with those of W = T/P
// threads of its row in the same wavefront (the row's T threads are T consecutive lanes, or
// every second lane of two rows side by side: ROWS 2), by a butterfly of cross-lane exchanges
// in a fixed order, stored by the first of them at num[row * P + j / W]. Where a wavefront
// holds 32 threads of each of two rows and W is 64, it sums both rows' in its one partial, the
// j / 32-th of the pair's 2P. The iteration's error sums them later in a fixed order too, so it
// stays deterministic; no block barrier is taken here.
// All lanes of the wavefront call it (store: whether this row exists; row0: the pair's first row).
template <int M, int T, int ROWS>
__device__ __forceinline__ void row_partials(double x, double* __restrict__ num, int row0, int c,
                                             int j, bool store) {
    constexpr int P = gs_partials_per_row(M), W = T / P;
    static_assert(W <= 64 && P * W == T, "partials of a row");
    constexpr bool PAIR = W * ROWS > 64;
#pragma unroll
    for (int o = 32; o > 0; o >>= 1)
        if (PAIR || (o >= ROWS && o < W * ROWS)) x += __shfl_xor(x, o, 64);
    if constexpr (PAIR) {
        if (store && c == 0 && (j & 31) == 0) num[(size_t)row0 * P + j / 32] = x;
    } else {
        if (store && (j & (W - 1)) == 0) num[(size_t)(row0 + c) * P + j / W] = x;
    }
}

// u -> a u/|u| (a where u = 0), u = scale * v; adds (|u| - a)^2 to acc.
__device__ __forceinline__ float2 constrain(float2 v, float scale, float a, double& acc) {
    const float re = v.x * scale, im = v.y * scale;
    const float m2 = re * re + im * im;
    const bool some = m2 > 0.f;  // (selects, not branches: the values of a row are independent)
    const float mag = some ? __fsqrt_rn(m2) : 0.f;
    const float f = a / mag;
    const double d = (double)mag - (double)a;
    acc += d * d;
    return make_float2(some ? re * f : a, some ? im * f : 0.f);
}

template <int M, bool HALF, class ST>
__global__ __launch_bounds__(RowCfg<M>::THREADS) void k_row_gs(
    typename ST::E* __restrict__ spec, const float* __restrict__ amp, float2* __restrict__ out,
    double* __restrict__ num, int nx, int ny, float scale, const float* __restrict__ dyn_inv,
    float fwd_scale, const float* __restrict__ dyn_fwd, const float2* __restrict__ tw) {
    using C = RowCfg<M>;
    using SE = typename ST::E;
    constexpr int E = C::E, T = C::T;
    __shared__ float2 lds[C::RPB * lds_elems<M>()];
    const int tid = threadIdx.x;
    const int sub = tid / T, j = tid % T;
    const int row = blockIdx.x * C::RPB + sub;
    const bool valid = row < ny;
    SE* srow = spec + (size_t)(valid ? row : 0) * M;
    const float* arow = amp + (size_t)(valid ? row : 0) * nx;
    float2* my_lds = lds + sub * lds_elems<M>();
    if (dyn_inv) scale *= *dyn_inv;
    TwCache<M, fused_of(ST::kFused, M), !ST::kFused> twc;
    twc.load(j, tw);
    float2 v[E];
#pragma unroll
    for (int r = 0; r < E; ++r)
        v[r] = valid ? ST::dec(srow[j + r * T]) : make_float2(0.f, 0.f);
    fft<M, INV>(v, my_lds, j, 0, twc);
    double acc = 0.0;
#pragma unroll
    for (int r = 0; r < E; ++r) {
        const int x = j + r * T;
        const bool in_field = HALF ? (r < E / 2) : (x < nx);
        if (in_field) {
            v[r] = constrain(v[r], scale, valid ? arow[x] : 0.f, acc);
        } else {
            v[r] = make_float2(0.f, 0.f);  // the padding of the next forward transform
        }
    }
    if (num) row_partials<M, T, 1>(acc, num, row, 0, j, valid);
    if (out) {
        if (valid) {
            float2* orow = out + (size_t)row * nx;
#pragma unroll
            for (int r = 0; r < E; ++r) {
                const int x = j + r * T;
                if (HALF ? (r < E / 2) : (x < nx)) orow[x] = v[r];
            }
        }
        return;
    }
    if (dyn_fwd) fwd_scale *= *dyn_fwd;
    if (fwd_scale != 1.0f) {
#pragma unroll
        for (int r = 0; r < E; ++r) v[r] = make_float2(v[r].x * fwd_scale, v[r].y * fwd_scale);
    }
    if constexpr (HALF) fft<M, FWD, 1, true>(v, my_lds, j, 0, twc);
    else fft<M, FWD>(v, my_lds, j, 0, twc);
    if (valid) {
#pragma unroll
        for (int r = 0; r < E; ++r) srow[j + r * T] = ST::enc(v[r]);
    }
}

// The same on the tiled spectrum plane (padded rows, Mx = 2Nx): two rows per block in
// neighbouring lanes, read and written as in k_row_inv_tile and k_row_fwd_tile (each block
// its own rows only).
template <int M, class ST>
__global__ __launch_bounds__(TileRowCfg<M>::THREADS) __attribute__((amdgpu_waves_per_eu(4))) void k_row_gs_tile(
    typename ST::E* __restrict__ spec, const float* __restrict__ amp, float2* __restrict__ out,
    double* __restrict__ num, int nx, int ny, float scale, const float* __restrict__ dyn_inv,
    float fwd_scale, const float* __restrict__ dyn_fwd, const float2* __restrict__ tw) {
    using C = TileRowCfg<M>;
    constexpr int E = kE, T = C::T, NL = E / 2;
    __shared__ float2 lds[C::LDS];
    const int c = threadIdx.x % C::ROWS, j = threadIdx.x / C::ROWS;
    if (dyn_inv) scale *= *dyn_inv;
    if (dyn_fwd) fwd_scale *= *dyn_fwd;
    const int y0 = xcd_remap(blockIdx.x, gridDim.x) * C::ROWS;
    const LayTile<typename ST::E> lay{ny};
    const unsigned at = lay.tile_lane(y0, j / kTileW, T / kTileW) + c * kTileW + j % kTileW;
    float2 v[E];
#pragma unroll
    for (int r = 0; r < E; ++r)
        v[r] = ST::dec((spec + lay.tile_step(y0, r * (T / kTileW), T / kTileW))[at]);
    TwCache<M, fused_of(ST::kFused, M), true> twc;
    twc.load(j, tw);
    fft<M, INV, C::ROWS>(v, lds, j, c, twc);
    // opaque copies of j: addresses and twiddles are made where they are used, not held
    int ja = j;
    asm volatile("" : "+v"(ja)::"memory");
    const size_t fy = (size_t)y0 * nx;
    const unsigned fx = (unsigned)c * nx + ja;
    float a[NL];
#pragma unroll
    for (int r = 0; r < NL; ++r) a[r] = (amp + fy + r * T)[fx];
    double acc = 0.0;
#pragma unroll
    for (int r = 0; r < NL; ++r) v[r] = constrain(v[r], scale, a[r], acc);
    if (num) row_partials<M, T, C::ROWS>(acc, num, y0, c, ja, true);
    if (out) {
#pragma unroll
        for (int r = 0; r < NL; ++r) (out + fy + r * T)[fx] = v[r];
        return;
    }
#pragma unroll
    for (int r = 0; r < NL; ++r) v[r] = make_float2(v[r].x * fwd_scale, v[r].y * fwd_scale);
    twc.j = ja;
    fft<M, FWD, C::ROWS, true>(v, lds, ja, c, twc);
    int jo = j;
    asm volatile("" : "+v"(jo)::"memory");
    const unsigned to = lay.tile_lane(y0, jo / kTileW, T / kTileW) + c * kTileW + jo % kTileW;
#pragma unroll
    for (int r = 0; r < E; ++r)
        (spec + lay.tile_step(y0, r * (T / kTileW), T / kTileW))[to] = ST::enc(v[r]);
}

// Rows of 2*MH as two transforms of MH each way (see rowsplit.hpp).
template <int MH, class ST>
__global__ __launch_bounds__(MH / 16 * kSplitRows) __attribute__((amdgpu_waves_per_eu(4))) void k_row_gs_tsplit(
    typename ST::E* __restrict__ spec, const float* __restrict__ amp, float2* __restrict__ out,
    double* __restrict__ num, int nx, int ny, float scale, const float* __restrict__ dyn_inv,
    float fwd_scale, const float* __restrict__ dyn_fwd, const float2* __restrict__ twm) {
    constexpr int E = kE, T = MH / E, R = kSplitRows;
    __shared__ float2 lds[R * lds_elems<MH>()];
    const int c = threadIdx.x % R, j = threadIdx.x / R;
    if (dyn_inv) scale *= *dyn_inv;
    if (dyn_fwd) fwd_scale *= *dyn_fwd;
    const int y0 = xcd_remap(blockIdx.x, gridDim.x) * R;
    const LayTile<typename ST::E> lay{ny};
    const unsigned at = lay.tile_lane(y0, j / 2, T / 2) + c * kTileW + 2 * (j & 1);
    using PK = Pack<typename ST::E, 2>;
    float2 ev[E], od[E];
#pragma unroll
    for (int r = 0; r < E; ++r) {
        const PK pk = *reinterpret_cast<const PK*>(spec + lay.tile_step(y0, r * (T / 2), T / 2) + at);
        ev[r] = ST::dec(pk.e[0]);
        od[r] = ST::dec(pk.e[1]);
    }
    TwCache<MH, ST::kFused, true> twc;
    twc.load_half(j, twm);
    fft<MH, INV, R>(od, lds, j, c, twc);
#pragma unroll
    for (int r = 0; r < E; ++r) {
        if (r % 4 == 0) asm volatile("" ::: "memory");
        od[r] = ctw<INV>(od[r], (twm + r * T)[j]);
    }
    asm volatile("" ::: "memory");
    fft<MH, INV, R>(ev, lds, j, c, twc);
    // opaque copies of j: addresses and twiddles are made where they are used, not held
    int ja = j;
    asm volatile("" : "+v"(ja)::"memory");
    const size_t fy = (size_t)y0 * nx;
    const unsigned fx = (unsigned)c * nx + ja;
#pragma unroll
    for (int r = 0; r < E; ++r) ev[r] = cadd(ev[r], od[r]);
    double acc = 0.0;
#pragma unroll
    for (int r = 0; r < E; ++r) {
        // four amplitudes at a time: the divisions in flight hold several registers each
        if (r % 4 == 0) asm volatile("" ::: "memory");
        ev[r] = constrain(ev[r], scale, (amp + fy + r * T)[fx], acc);
    }
    if (num) row_partials<2 * MH, T, R>(acc, num, y0, c, ja, true);
    if (out) {
#pragma unroll
        for (int r = 0; r < E; ++r) (out + fy + r * T)[fx] = ev[r];
        return;
    }
#pragma unroll
    for (int r = 0; r < E; ++r) ev[r] = od[r] = make_float2(ev[r].x * fwd_scale, ev[r].y * fwd_scale);
    twc.j = ja;
    fft<MH, FWD, R>(ev, lds, ja, c, twc);
    int jo = j;
    asm volatile("" : "+v"(jo)::"memory");
    twc.j = jo;
#pragma unroll
    for (int r = 0; r < E; ++r) od[r] = cmul(od[r], (twm + r * T)[jo]);
    fft<MH, FWD, R>(od, lds, jo, c, twc);
    const unsigned to = lay.tile_lane(y0, jo / 2, T / 2) + c * kTileW + 2 * (jo & 1);
#pragma unroll
    for (int r = 0; r < E; ++r) {
        const PK pk{{ST::enc(ev[r]), ST::enc(od[r])}};
        *reinterpret_cast<PK*>(spec + lay.tile_step(y0, r * (T / 2), T / 2) + to) = pk;
    }
}

// Sum of f(v[i]) in FP64 over i = lo + threadIdx.x, + step, ... < hi, eight loads in flight, in
// the order of i (f's values are added one by one).
template <class V, class F>
__device__ __forceinline__ double strided_sum(const V* __restrict__ v, long long lo, long long hi,
                                              int step, F f) {
    constexpr int U = 8;
    double t = 0.0;
    long long i = lo + threadIdx.x;
    for (; i + (U - 1) * step < hi; i += U * step) {
        V x[U];
#pragma unroll
        for (int k = 0; k < U; ++k) x[k] = v[i + k * step];
#pragma unroll
        for (int k = 0; k < U; ++k) t += f(x[k]);
    }
    for (; i < hi; i += step) t += f(v[i]);
    return t;
}

// Sum over a block of NT threads by a fixed tree; every thread gets the result.
template <int NT>
__device__ __forceinline__ double block_sum(double t) {
    __shared__ double red[NT / 64];
#pragma unroll
    for (int d = 32; d > 0; d >>= 1) t += __shfl_xor(t, d);
    __syncthreads();
    if (threadIdx.x % 64 == 0) red[threadIdx.x / 64] = t;
    __syncthreads();
    double r = 0.0;
#pragma unroll
    for (int w = 0; w < NT / 64; ++w) r += red[w];
    return r;
}

// den = sum(amp^2) in FP64 as kGsDenParts partials, partial b over the contiguous chunk b
// of the array: the same order on every run. (1024^2 and 2048^2 values on average 4.7 us, with
// one load in flight per thread 7.3.)
__global__ __launch_bounds__(256) void k_gs_den(const float* __restrict__ amp,
                                                double* __restrict__ part, long long count) {
    const long long chunk = (count + gridDim.x - 1) / gridDim.x;
    const long long lo = (long long)blockIdx.x * chunk;
    const long long hi = lo + chunk < count ? lo + chunk : count;
    const double t = block_sum<256>(strided_sum(amp, lo, hi, 256, [](float a) { return (double)a * a; }));
    if (threadIdx.x == 0) part[blockIdx.x] = t;
}

// iteration k's error from its n = ny * P row partials and the denominator's partials,
// each summed in a fixed order. One block per iteration, so as many threads and loads in flight as
// a block can have (4096 and 16384 partials on average 4.8 us, with 256 threads
// and one load each 12.9).
constexpr int kGsErrThreads = 1024;
__global__ __launch_bounds__(kGsErrThreads) void k_gs_errors(const double* __restrict__ num,
                                                             const double* __restrict__ den_part,
                                                             float* __restrict__ errors, int n) {
    const auto same = [](double x) { return x; };
    const int k = blockIdx.x;
    const double tn = strided_sum(num + (size_t)k * n, 0, n, kGsErrThreads, same);
    const double td = strided_sum(den_part, 0, kGsDenParts, kGsErrThreads, same);
    const double sn = block_sum<kGsErrThreads>(tn);
    const double sd = block_sum<kGsErrThreads>(td);
    if (threadIdx.x == 0) errors[k] = (float)sqrt(sn / sd);
}

// ---- host launchers ------------------------------------------------------------

namespace {
template <class ST>
hipError_t row_gs_t(void* spec, const float* amp, float2* out, double* num, int nx, int ny,
                    int mx, float scale, const float* dyn_inv, float fwd_scale,
                    const float* dyn_fwd, const float2* tw, hipStream_t s, int layout) {
    using SE = typename ST::E;
    const bool half = (mx == 2 * nx);
    if (layout == 1) {
        if (!half) return hipErrorInvalidValue;
        CWO_DISPATCH_M(mx, {
            if constexpr (MM == 8192 && ST::kFused) {
                launch_kernel((k_row_gs_tsplit<MM / 2, ST>), dim3(ny / kSplitRows),
                                   dim3(MM / 32 * kSplitRows), 0, s, (SE*)spec, amp, out, num, nx, ny,
                                   scale, dyn_inv, fwd_scale, dyn_fwd, tw);
            } else if constexpr (MM >= 512 && MM <= 4096) {
                using C = TileRowCfg<MM>;
                launch_kernel((k_row_gs_tile<MM, ST>), dim3(ny / C::ROWS), dim3(C::THREADS), 0, s,
                                   (SE*)spec, amp, out, num, nx, ny, scale, dyn_inv, fwd_scale,
                                   dyn_fwd, tw);
            } else {
                return hipErrorInvalidValue;
            }
        });
        return hipGetLastError();
    }
    CWO_DISPATCH_M(mx, {
        using C = RowCfg<MM>;
        dim3 grid((ny + C::RPB - 1) / C::RPB);
        if (half)
            launch_kernel((k_row_gs<MM, true, ST>), grid, dim3(C::THREADS), 0, s, (SE*)spec,
                               amp, out, num, nx, ny, scale, dyn_inv, fwd_scale, dyn_fwd, tw);
        else
            launch_kernel((k_row_gs<MM, false, ST>), grid, dim3(C::THREADS), 0, s, (SE*)spec,
                               amp, out, num, nx, ny, scale, dyn_inv, fwd_scale, dyn_fwd, tw);
    });
    return hipGetLastError();
}
}  // namespace

hipError_t launch_row_gs(void* spec, const float* amp, float2* out, double* num, int nx, int ny,
                         int mx, const GsScale& gsc, const float2* tw, hipStream_t s) {
    switch (gsc.prec) {
        case 0:
            return row_gs_t<StF32>(spec, amp, out, num, nx, ny, mx, gsc.scale, gsc.dyn_inv,
                                   gsc.fwd_scale, gsc.dyn_fwd, tw, s, gsc.layout);
        case 1:
            return row_gs_t<StF16>(spec, amp, out, num, nx, ny, mx, gsc.scale, gsc.dyn_inv,
                                   gsc.fwd_scale, gsc.dyn_fwd, tw, s, gsc.layout);
        case 2:
            return row_gs_t<StBF16>(spec, amp, out, num, nx, ny, mx, gsc.scale, gsc.dyn_inv,
                                    gsc.fwd_scale, gsc.dyn_fwd, tw, s, gsc.layout);
    }
    return hipErrorInvalidValue;
}

int gs_partials(int mx) { return gs_partials_per_row(mx); }

hipError_t launch_gs_errors(const double* num, const float* amp, double* den_work, float* errors,
                            int nx, int ny, int mx, int iters, hipStream_t s) {
    launch_kernel(k_gs_den, dim3(kGsDenParts), dim3(256), 0, s, amp, den_work, (long long)nx * ny);
    launch_kernel(k_gs_errors, dim3(iters), dim3(kGsErrThreads), 0, s, num, (const double*)den_work,
                       errors, ny * gs_partials_per_row(mx));
    return hipGetLastError();
}

}  // namespace cwo
