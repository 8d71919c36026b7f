// Column pass of the diffraction path: forward FFT along y, multiplication by the
// transfer function generated per bin, inverse FFT, crop (shared by the plain, shifted
// and ping-pong forms).
#pragma once
#include "kernel_common.hpp"

namespace cwo {

// ---- column pass: FFT, transfer function, IFFT, crop --------------------------

// Exact form, for any parameters: per bin in FP64, the propagating test s <= 1 evaluated
// as lam*(p'*df) squared and summed, each operation rounded on its own (fused
// multiply-adds are switched off, so the decision is that of the plain FP64 definition),
// sine/cosine of the reduced phase in FP32.
struct AsmH {
    double dfx, dfy;  // frequency pitches 1/(Mx dx), 1/(My dy)
    double lam;       // wavelength
    double zl;        // z / lambda: phase in revolutions per unit sqrt(1 - s)
    int mx, my;
    struct Col {
        double ax2;
    };
    __device__ __forceinline__ Col column(int p) const {
#pragma clang fp contract(off)
        const double pp = (double)(p < mx / 2 ? p : p - mx);
        const double ax = lam * (pp * dfx);
        return Col{ax * ax};
    }
    struct Row {
        double ay2;
    };
    __device__ __forceinline__ Row row(const Col&, int j, int, int soff) const {
#pragma clang fp contract(off)
        const double qq = (double)(j + soff);
        const double ay = lam * (qq * dfy);
        return Row{ay * ay};
    }
    __device__ __forceinline__ float2 operator()(const Col& c, const Row& rw) const {
#pragma clang fp contract(off)
        // s = (lambda*fx)^2 + (lambda*fy)^2 with fx = p'*dfx, evaluated without contraction
        const double s = rw.ay2 + c.ax2;
        if (!(s <= 1.0)) return make_float2(0.f, 0.f);  // evanescent bin
        const double t = zl * sqrt(1.0 - s);             // revolutions
        const float r = (float)(t - rint(t));            // [-0.5, 0.5]
        return make_float2(__builtin_amdgcn_cosf(r), __builtin_amdgcn_sinf(r));
    }
};

// Fast form, used when every bin has s = (lambda fx)^2 + (lambda fy)^2 <= 0.05 (so none is
// evanescent): with x = s/2, 1 - sqrt(1 - 2x) = x + x^2/2 + x^3/2 + 5x^4/8 + ..., so the phase
// in revolutions is zl - zl*(x + ...), evaluated in FP64 with its sign turned, zl in the
// coefficients and the constant reduced on the host, and reduced to [-1/2, 1/2] in FP64 before
// it is rounded to FP32: the phases of z and -z are then rounded alike, so that a propagation
// there and back cancels them (the ping-pong iteration of 512^2: 2.4e-7 off, with the fraction in
// [0, 1), one operation less, 4.4e-7). The series to n = 9 has a truncation error below 3e-12
// relative for s <= 0.05, and the launcher takes NT = 4 where zl times the rest of the series is
// below 2^-28 revolution on the whole grid. The hardware sine and cosine take revolutions. One
// series for the whole phase costs a bin six FP64 multiply-adds; reducing column, row and
// remainder terms separately took eight FP64 and three FP32 operations.
template <int NT>
struct AsmHFastN {
    static_assert(NT == 4 || NT == 9, "series length");
    double hdx, hdy;  // lambda/(Mx dx), lambda/(My dy), both over sqrt(2)
    double k0, k1;    // -zl reduced to [-0.5, 0.5]; zl = z/lambda
    double k23, k4;   // zl/2, 5 zl/8
    int mx, my;
    void set(double lam_dfx, double lam_dfy, double zl, double minus_zl_reduced) {
        hdx = lam_dfx * 0.70710678118654752440;
        hdy = lam_dfy * 0.70710678118654752440;
        k0 = minus_zl_reduced;
        k1 = zl;
        k23 = 0.5 * zl;
        k4 = 0.625 * zl;
    }
    struct Col {
        double a, k4, dy;
    };
    __device__ __forceinline__ Col column(int p) const {
        const double x = (double)(p < mx / 2 ? p : p - mx) * hdx;
        // in vector registers: a multiply-add takes one scalar operand at most
        double c4 = k4, dy = hdy;
        asm("" : "+v"(c4), "+v"(dy));
        return Col{x * x, c4, dy};
    }
    struct Row {
        double y;
    };
    __device__ __forceinline__ Row row(const Col& c, int j, int, int soff) const {
        return Row{fma((double)soff, c.dy, (double)j * c.dy)};
    }
    // minus the phase in revolutions
    __device__ __forceinline__ double turns(const Col& c, const Row& rw) const {
        const double x = fma(rw.y, rw.y, c.a);
        double q = c.k4;
        if constexpr (NT == 9) {
            double t = 5.5859375;
            t = fma(t, x, 3.3515625);
            t = fma(t, x, 2.0625);
            t = fma(t, x, 1.3125);
            t = fma(t, x, 0.875);
            q = fma(k1 * t, x, q);
        }
        q = fma(q, x, k23);
        q = fma(q, x, k23);
        q = fma(q, x, k1);
        return fma(q, x, k0);
    }
    __device__ __forceinline__ float2 operator()(const Col& c, const Row& rw) const {
        const double t = turns(c, rw);
        const float r = (float)(t - rint(t));
        return make_float2(__builtin_amdgcn_cosf(r), -__builtin_amdgcn_sinf(r));
    }
};
using AsmHFast = AsmHFastN<9>;

// The same for 16-bit storage (see kFused), in the terms its stored planes are made from: with
// T(s) = 1 - s/2 - sqrt(1 - s), the phase splits exactly into
//     (z/lambda) sqrt(1 - s) = zl - zl*a/2 - zl*b/2 - zl*T(s),  s = a + b,
// a = (lambda fx)^2 per column, b = (lambda fy)^2 per row, every large term reduced modulo one
// revolution in FP64 before it is rounded to FP32.
template <int NT>
struct AsmHFast16N {
    static_assert(NT == 4 || NT == 9, "series length");
    double lam_dfx, lam_dfy;  // lambda/(Mx dx), lambda/(My dy)
    double zl, half_zl;       // z/lambda, z/(2 lambda)
    float c0;                 // zl reduced to [-0.5, 0.5]
    int mx, my;
    void set(double ldx, double ldy, double z, double minus_zl_reduced) {
        lam_dfx = ldx;
        lam_dfy = ldy;
        zl = z;
        half_zl = 0.5 * z;
        c0 = (float)-minus_zl_reduced;
    }
    struct Col {
        double a;
        float ca;  // c0 - reduced(zl*a/2)
    };
    __device__ __forceinline__ Col column(int p) const {
        const double x = (double)(p < mx / 2 ? p : p - mx) * lam_dfx;
        const double a = x * x;
        const double ta = half_zl * a;
        return Col{a, c0 - (float)(ta - rint(ta))};
    }
    struct Row {
        double b, hb;  // (lambda fy)^2 and zl*b/2
    };
    __device__ __forceinline__ Row row(const Col&, int j, int, int soff) const {
        const double y = (double)(j + soff) * lam_dfy;
        const double b = y * y;
        return Row{b, half_zl * b};
    }
    __device__ __forceinline__ float2 operator()(const Col& c, const Row& rw) const {
        const double s = c.a + rw.b;
        double poly;
        if constexpr (NT == 9) {
            poly = 715.0 / 65536.0;
            poly = fma(poly, s, 429.0 / 32768.0);
            poly = fma(poly, s, 33.0 / 2048.0);
            poly = fma(poly, s, 21.0 / 1024.0);
            poly = fma(poly, s, 7.0 / 256.0);
            poly = fma(poly, s, 5.0 / 128.0);
        } else {
            poly = 5.0 / 128.0;
        }
        poly = fma(poly, s, 1.0 / 16.0);
        poly = fma(poly, s, 1.0 / 8.0);
        // zl*b/2 + zl*T(s), reduced (the exact fractional part), in FP64
        const double u = fma(zl * (s * s), poly, rw.hb);
        float r = c.ca - (float)__builtin_amdgcn_fract(u);
        r -= rintf(r);
        return make_float2(__builtin_amdgcn_cosf(r), __builtin_amdgcn_sinf(r));
    }
};


struct FresnelH {
    const float2* __restrict__ hx;  // Mx entries, carries the constant C
    const float2* __restrict__ hy;  // My entries
    struct Col {
        float2 h;
    };
    struct Row {
        float2 h;
    };
    __device__ __forceinline__ Col column(int p) const { return Col{hx[p]}; }
    __device__ __forceinline__ Row row(const Col&, int j, int off, int) const {
        return Row{(hy + off)[j]};
    }
    __device__ __forceinline__ float2 operator()(const Col& c, const Row& rw) const {
        return cmul(c.h, rw.h);
    }
};

// ---- per-plane transfer functions of a mixed batch -------------------------------------
//
// Planes of one geometry (sizes, pitch, flags) whose distance, wavelength or kind differ
// share the row passes; their column pass runs as one launch per transfer-function form
// present (fast ASM with the series to s^4, to s^9, Fresnel factors), each over its planes
// listed by buffer index, and each plane gets exactly the transfer function its single call
// would use. The kernel of each form is the single-plane kernel of that form.
template <class HF>
struct PlaneList {
    int n;
    int idx[kZChunk];  // buffer plane of launch plane k
    HF f[kZChunk];     // its transfer function
};

// Transfer function and buffer plane of launch plane pl: the functor itself and pl, or the
// list's entries.
template <class HF>
__device__ __forceinline__ const HF& plane_tf(const HF& hf, int) {
    return hf;
}
template <class HF>
__device__ __forceinline__ const HF& plane_tf(const PlaneList<HF>& t, int pl) {
    return t.f[pl];
}
template <class HF>
__device__ __forceinline__ int buffer_plane(const HF&, int pl) {
    return pl;
}
template <class HF>
__device__ __forceinline__ int buffer_plane(const PlaneList<HF>& t, int pl) {
    return t.idx[pl];
}

// Waves per SIMD the column kernels are compiled for: four (128 VGPRs), where the fast forms
// spill nothing below columns of 8192. The exact forms hold FP64 values beside the column and spill 8 to
// 145 registers there; with two waves none, which is faster except for complex64 columns of 4096
// at full length, whose blocks of 512 threads then have a CU each. Four and two waves, planes of
// the exact form: 512^2 complex64 20.6 and 19.6 us, 2048^2 98.6 and 119, 4096^2 517 and 507; FP16
// 1024^2 42.3 and 39.4, 2048^2 142 and 126, 4096^2 595 and 493; shifted 4096^2 686 and 561, FP16
// 725 and 539.
template <class HF>
constexpr bool kExactForm = false;
template <>
inline constexpr bool kExactForm<AsmH> = true;
template <class HF, class ST, int M, bool SPLIT>
constexpr int col_waves() {
    return kExactForm<HF> && !(M == 4096 && !SPLIT && std::is_same_v<ST, StF32>) ? 2 : 4;
}

// Transfer function objects give column(p) for a column and row(column, j, off, soff) for its
// row j + off, soff being off as a signed frequency index offset (off or off - My).

// Column pass: forward FFT of COLS columns, multiplication by the transfer function,
// inverse FFT, in place; one (plane, column tile) item per block. LAY addresses the
// plane (row-major or tiled). With HALF the rows Ny..My-1 of the padded column are zero:
// they are neither loaded nor added in the first forward pass, and only rows < Ny of the
// result are computed to the end and stored. hscale (a power of two; complex64 storage has
// none) multiplies the stored values; scaling by a power of two commutes exactly with
// the inverse transform, so this equals scaling the transfer function.
template <int M, bool HALF, class HF, class ST, class LAY>
__global__ __launch_bounds__(ColCfg<M>::THREADS) __attribute__((amdgpu_waves_per_eu(col_waves<HF, ST, M, false>()))) void k_col(typename ST::E* __restrict__ buf,
                                                              int ny, int mx, int batch,
                                                              size_t plane, HF hf, float hscale,
                                                              const float2* __restrict__ tw,
                                                              LAY lay) {
    using C = ColCfg<M>;
    constexpr int E = kE, T = C::T;
    using SE = typename ST::E;
    __shared__ float2 lds[C::LDS];
    const int c = threadIdx.x % C::COLS, j = threadIdx.x / C::COLS;
    const int ntiles = (mx + C::COLS - 1) / C::COLS;
    const int it = xcd_remap(blockIdx.x, gridDim.x);
    const int pl = it / ntiles, tile = it - pl * ntiles;
    const int col0 = tile * C::COLS + c;
    // tiles may overhang planes narrower than a tile
    const bool active = C::COLS <= 16 || col0 < mx;
    const int col = active ? col0 : 0;
    SE* base = buf + buffer_plane(hf, pl) * plane;
    const auto& hfp = plane_tf(hf, pl);  // this block's transfer function
    using PH = std::decay_t<decltype(hfp)>;
    const int lt = C::COLS <= kTileW ? tile * C::COLS / kTileW : col / kTileW;  // layout tile
    const unsigned at = lay.lane(j, col, lt, T);
    float2 v[E];
#pragma unroll
    for (int r = 0; r < E; ++r) {
        const bool ld = active && (HALF ? (r < E / 2) : (j + r * T < ny));
        v[r] = ld ? ST::dec((base + lay.step(r * T, lt, T))[at]) : make_float2(0.f, 0.f);
    }
    // (the 16 factors of the two-step passes fit beside 4096-point columns only)
    TwCache<M, fused_of(ST::kFused, M), !ST::kFused && M != 4096> twc;
    twc.load(j, tw);
    const typename PH::Col hc = hfp.column(col);
    fft<M, FWD, C::COLS, HALF>(v, lds, j, c, twc);
    fft_mul<M, INV, C::COLS>(
        v,
        [&](auto rc) {
            constexpr int r = decltype(rc)::value, off = r * T;
            return hfp(hc, hfp.row(hc, j, off, off < M / 2 ? off : off - M));
        },
        lds, j, c, twc);
#pragma unroll
    for (int r = 0; r < E; ++r) {
        const bool st = active && (HALF ? (r < E / 2) : (j + r * T < ny));
        if constexpr (!std::is_same_v<ST, StF32>) v[r] = make_float2(v[r].x * hscale, v[r].y * hscale);
        if (st) (base + lay.step(r * T, lt, T))[at] = ST::enc(v[r]);
    }
}

// Column pass for padded columns of length M = 2*MH with MH non-zero rows, as two
// transforms of length MH. With W = exp(-2 pi i/M), the padded forward transform's even
// bins are DFT_MH(x)[k] and its odd bins DFT_MH(x_n W^n)[k]; after multiplying by H(2k) and
// H(2k+1), the first MH outputs of the padded inverse transform are
// IDFT_MH(even)[n] + W^-n IDFT_MH(odd)[n]. Two columns per block in neighbouring lanes, as in
// the full-length kernel; a thread does the even and the odd bins of its column one after the
// other, so that it keeps to 128 VGPRs (the column or the even bins' result, the values in
// work and one pass's twiddles) and a block to the LDS of one transform per column.
// twm: the length-M table.
template <int MH, class HF, class ST, class LAY>
__global__ __launch_bounds__(MH / 8) __attribute__((amdgpu_waves_per_eu(col_waves<HF, ST, 2 * MH, true>()))) void k_col_split(
    typename ST::E* __restrict__ buf, int ny, int mx, int batch, size_t plane, HF hf, float hscale,
    const float2* __restrict__ twm, LAY lay) {
    constexpr int E = kE, T = MH / E, C = 2;
    using SE = typename ST::E;
    __shared__ float2 lds[C * lds_elems<MH>()];
    const int c = threadIdx.x % C, j = threadIdx.x / C;
    const int ntiles = mx / C;
    const int it = xcd_remap(blockIdx.x, gridDim.x);
    const int pl = it / ntiles, tile = it - pl * ntiles, col = tile * C + c;
    SE* base = buf + buffer_plane(hf, pl) * plane;
    const auto& hfp = plane_tf(hf, pl);
    using PH = std::decay_t<decltype(hfp)>;
    const int lt = tile * C / kTileW;  // layout tile
    const unsigned at = lay.lane(j, col, lt, T);
    float2 ev[E], od[E];
#pragma unroll
    for (int r = 0; r < E; ++r) ev[r] = od[r] = ST::dec((base + lay.step(r * T, lt, T))[at]);
    TwCache<MH, ST::kFused, true> twc;
    twc.load_half(j, twm);
    const typename PH::Col hc = hfp.column(col);
    auto filter = [&](float2 (&v)[E], int j, int odd) {
        fft<MH, FWD, C>(v, lds, j, c, twc);
        fft_mul<MH, INV, C>(
            v,
            [&](auto rc) {
                constexpr int r = decltype(rc)::value, off = 2 * r * T;
                return hfp(hc, hfp.row(hc, 2 * j + odd, off, off < MH ? off : off - 2 * MH));
            },
            lds, j, c, twc);
    };
    filter(ev, j, 0);
    // opaque copies of j: addresses and twiddles are made where they are used, not held
    int jo = j;
    asm volatile("" : "+v"(jo)::"memory");
#pragma unroll
    for (int r = 0; r < E; ++r) od[r] = cmul(od[r], (twm + r * T)[jo]);
    twc.j = jo;
    filter(od, jo, 1);
    int js = j;
    asm volatile("" : "+v"(js)::"memory");
    const unsigned as = lay.lane(js, col, lt, T);
#pragma unroll
    for (int r = 0; r < E; ++r) {
        float2 o = cadd(ev[r], ctw<INV>(od[r], (twm + r * T)[js]));
        if constexpr (!std::is_same_v<ST, StF32>) o = make_float2(o.x * hscale, o.y * hscale);
        (base + lay.step(r * T, lt, T))[as] = ST::enc(o);
    }
}

}  // namespace cwo
