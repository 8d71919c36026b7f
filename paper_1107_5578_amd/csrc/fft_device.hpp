// Device-side FFT building blocks for gfx950 (wave64, LDS-staged Stockham).
//
// A length-M transform is done by one group of T = M/16 threads; each thread
// holds 16 complex values in registers. Before every pass thread j holds the
// elements j + r*T (r < 16) of the current sequence; a radix-RP pass performs
// 16/RP butterflies b = j + i*T, each reading inputs b + kk*(M/RP), multiplying
// by the Stockham twiddle W_{Ns*RP}^{(b mod Ns)*kk} and writing outputs to
// (b / Ns)*Ns*RP + (b mod Ns) + kk*Ns, where Ns is the product of the radices
// of the earlier passes. The first pass takes the remaining radix 2, 4, 8 (or 16), every
// later one is of radix 16. Intermediate passes exchange through LDS; the first
// pass reads registers loaded straight from global memory and the last pass
// leaves the result in registers in natural order (element j + r*T), so global
// loads and stores are both unit-stride across a wavefront.
//
// Sign convention: forward uses exp(-2*pi*i*jk/M), inverse exp(+2*pi*i*jk/M),
// both unnormalised (the DFT pair the paper's FFT/IFFT primitives compute).
#pragma once
#include <hip/hip_runtime.h>

#include <utility>

#include "launch.hpp"

namespace cwo {

constexpr int FWD = -1;
constexpr int INV = +1;

// ---- storage of the padded intermediate planes --------------------------------
// complex64 (FP32), or two FP16 / two BF16 values per complex (rounded to nearest
// even on the way in). Arithmetic is always FP32.
//
// kFused says which of the two transform arithmetics a storage takes: the fused one for
// complex64 (from kFusedMin points on, see fused_of); the two-step one for 16-bit storage,
// whose roundings turn a last-bit change of an FP32 value into half a unit of 16 bits, so that
// its stored planes stay the values they were before the fused arithmetic existed.
struct StF32 {
    static constexpr bool kFused = true;
    using E = float2;
    __device__ __forceinline__ static float2 dec(E v) { return v; }
    __device__ __forceinline__ static E enc(float2 v) { return v; }
};
struct alignas(4) half2s {
    _Float16 x, y;
};
struct StF16 {
    static constexpr bool kFused = false;
    using E = half2s;
    __device__ __forceinline__ static float2 dec(E v) { return make_float2((float)v.x, (float)v.y); }
    __device__ __forceinline__ static E enc(float2 v) { return E{(_Float16)v.x, (_Float16)v.y}; }
};
struct alignas(4) bf162s {
    __bf16 x, y;
};
struct StBF16 {
    static constexpr bool kFused = false;
    using E = bf162s;
    __device__ __forceinline__ static float2 dec(E v) { return make_float2((float)v.x, (float)v.y); }
    __device__ __forceinline__ static E enc(float2 v) { return E{(__bf16)v.x, (__bf16)v.y}; }
};
// P adjacent stored elements, loaded and stored as one vector access
template <class E, int P>
struct alignas(sizeof(E) * P) Pack {
    E e[P];
};

__device__ __forceinline__ float2 cadd(float2 a, float2 b) { return make_float2(a.x + b.x, a.y + b.y); }
__device__ __forceinline__ float2 csub(float2 a, float2 b) { return make_float2(a.x - b.x, a.y - b.y); }
__device__ __forceinline__ float2 cmul(float2 a, float2 b) {
    return make_float2(__fmaf_rn(a.x, b.x, -a.y * b.y), __fmaf_rn(a.x, b.y, a.y * b.x));
}
// multiply by w (DIR = FWD) or conj(w) (DIR = INV); tables store exp(-2*pi*i*k/M)
template <int DIR>
__device__ __forceinline__ float2 ctw(float2 a, float2 w) {
    if constexpr (DIR == FWD) return cmul(a, w);
    else return make_float2(__fmaf_rn(a.x, w.x, a.y * w.y), __fmaf_rn(a.y, w.x, -a.x * w.y));
}
// multiply by exp(DIR * i*pi/2): -i forward, +i inverse
template <int DIR>
__device__ __forceinline__ float2 rot90(float2 a) {
    if constexpr (DIR == FWD) return make_float2(a.y, -a.x);
    else return make_float2(-a.y, a.x);
}

// Multiply by exp(DIR * 2*pi*i*m/R) for a compile-time m, cheap forms for multiples of pi/4.
template <int R, int M_, int DIR>
__device__ __forceinline__ float2 wconst(float2 a) {
    constexpr int m = ((M_ % R) + R) % R;
    if constexpr (m == 0) return a;
    else if constexpr (8 * m % R == 0) {
        constexpr int oct = 8 * m / R;  // angle = oct * pi/4
        constexpr float h = 0.70710678118654752440f;
        if constexpr (oct == 2) return rot90<DIR>(a);
        else if constexpr (oct == 4) return make_float2(-a.x, -a.y);
        else if constexpr (oct == 6) return rot90<-DIR>(a);
        else {
            // (+-1 +- i)/sqrt(2): angle = DIR*oct*pi/4
            constexpr float c = (oct == 1 || oct == 7) ? h : -h;
            constexpr float s0 = (oct == 1 || oct == 3) ? h : -h;  // sin(oct*pi/4)
            constexpr float s = (DIR == FWD) ? -s0 : s0;
            // fused as in the general case, so that every kernel rounds it alike
            return make_float2(__fmaf_rn(c, a.x, -s * a.y), __fmaf_rn(c, a.y, s * a.x));
        }
    } else {
        // general angle 2*pi*m/R with R <= 32: cos/sin of multiples of pi/16
        constexpr double PI = 3.14159265358979323846;
        // constexpr evaluation through a small table of cos(k*pi/16), k = 0..8
        constexpr double ctab[9] = {1.0, 0.98078528040323044913, 0.92387953251128675613,
                                    0.83146961230254523708, 0.70710678118654752440,
                                    0.55557023301960222474, 0.38268343236508977173,
                                    0.19509032201612826785, 0.0};
        constexpr int k32 = m * (32 / R);  // angle in units of pi/16, 0..31
        constexpr int q = k32 / 8, rr = k32 % 8;
        // cos and sin of (q*pi/2 + rr*pi/16)
        constexpr double c0 = ctab[rr], s0 = ctab[8 - rr];
        constexpr double cc = q == 0 ? c0 : q == 1 ? -s0 : q == 2 ? -c0 : s0;
        constexpr double ss = q == 0 ? s0 : q == 1 ? c0 : q == 2 ? -s0 : -c0;
        constexpr float c = (float)cc;
        constexpr float s = (float)(DIR == FWD ? -ss : ss);
        (void)PI;
        return make_float2(__fmaf_rn(c, a.x, -s * a.y), __fmaf_rn(c, a.y, s * a.x));
    }
}

// ---- two-step arithmetic: twiddle each input, then a DFT of 4 x 4 points ----------
//
// Small DFTs on register arrays, in place, natural output order.

template <int DIR>
__device__ __forceinline__ void dft2(float2& a, float2& b) {
    float2 t = a;
    a = cadd(t, b);
    b = csub(t, b);
}

template <int DIR>
__device__ __forceinline__ void dft4(float2& a0, float2& a1, float2& a2, float2& a3) {
    float2 t0 = cadd(a0, a2), t1 = csub(a0, a2);
    float2 t2 = cadd(a1, a3), t3 = rot90<DIR>(csub(a1, a3));
    a0 = cadd(t0, t2);
    a2 = csub(t0, t2);
    a1 = cadd(t1, t3);
    a3 = csub(t1, t3);
}

// DFT of 4 points of which the last two are zero: 8 additions instead of 16.
template <int DIR>
__device__ __forceinline__ void dft4_zin(float2& a0, float2& a1, float2& a2, float2& a3) {
    const float2 x0 = a0, x1 = a1, r = rot90<DIR>(a1);
    a0 = cadd(x0, x1);
    a2 = csub(x0, x1);
    a1 = cadd(x0, r);
    a3 = csub(x0, r);
}

// DFT of R points held in v[OFF + STRIDE*k], k < R, result in the same slots in natural order.
// ZIN: the inputs k >= R/2 are known to be zero (the zero-padded half of a transform's
// first pass) and are neither read nor added; each half-size DFT of the decimation in
// time then has a zero upper half as well.
template <int R, int DIR, int OFF = 0, int STRIDE = 1, bool ZIN = false, int N>
__device__ __forceinline__ void dft(float2 (&v)[N]) {
    static_assert(R == 1 || R == 2 || R == 4 || R == 8 || R == 16, "radix");
    if constexpr (R == 1) {
        return;
    } else if constexpr (R == 2) {
        if constexpr (ZIN) v[OFF + STRIDE] = v[OFF];
        else dft2<DIR>(v[OFF], v[OFF + STRIDE]);
    } else if constexpr (R == 4) {
        if constexpr (ZIN) dft4_zin<DIR>(v[OFF], v[OFF + STRIDE], v[OFF + 2 * STRIDE], v[OFF + 3 * STRIDE]);
        else dft4<DIR>(v[OFF], v[OFF + STRIDE], v[OFF + 2 * STRIDE], v[OFF + 3 * STRIDE]);
    } else if constexpr (R == 8) {
        // radix-2 decimation in time over two half-size DFTs
        constexpr int H = R / 2;
        dft<H, DIR, OFF, 2 * STRIDE, ZIN>(v);           // even samples
        dft<H, DIR, OFF + STRIDE, 2 * STRIDE, ZIN>(v);  // odd samples
        float2 t[R];
#pragma unroll
        for (int k = 0; k < R; ++k) t[k] = v[OFF + k * STRIDE];
        // t[2k] = E[k], t[2k+1] = O[k]
        float2 o[R];
        [&]<int... K>(std::integer_sequence<int, K...>) {
            ((o[K] = cadd(t[2 * K], wconst<R, K, DIR>(t[2 * K + 1])),
              o[K + H] = csub(t[2 * K], wconst<R, K, DIR>(t[2 * K + 1]))), ...);
        }(std::make_integer_sequence<int, H>{});
#pragma unroll
        for (int k = 0; k < R; ++k) v[OFF + k * STRIDE] = o[k];
    } else {  // R == 16: 4 x 4
        // stage 1: for each n2, DFT4 over n1 of x[4*n1 + n2]; result Y[n2][k1] kept at slot 4*k1 + n2
        // (with ZIN, x[4*n1 + n2] = 0 for n1 >= 2)
        dft<4, DIR, OFF + 0 * STRIDE, 4 * STRIDE, ZIN>(v);
        dft<4, DIR, OFF + 1 * STRIDE, 4 * STRIDE, ZIN>(v);
        dft<4, DIR, OFF + 2 * STRIDE, 4 * STRIDE, ZIN>(v);
        dft<4, DIR, OFF + 3 * STRIDE, 4 * STRIDE, ZIN>(v);
        // twiddles W16^(n2*k1) on slot 4*k1 + n2
        float2 y[16];
        [&]<int... S>(std::integer_sequence<int, S...>) {
            ((y[S] = wconst<16, (S % 4) * (S / 4), DIR>(v[OFF + S * STRIDE])), ...);
        }(std::make_integer_sequence<int, 16>{});
        // stage 2: for each k1, DFT4 over n2 of Y[n2][k1] -> X[k1 + 4*k2]
        dft4<DIR>(y[0], y[1], y[2], y[3]);
        dft4<DIR>(y[4], y[5], y[6], y[7]);
        dft4<DIR>(y[8], y[9], y[10], y[11]);
        dft4<DIR>(y[12], y[13], y[14], y[15]);
        // y[4*k1 + k2] = X[k1 + 4*k2]
#pragma unroll
        for (int k1 = 0; k1 < 4; ++k1)
#pragma unroll
            for (int k2 = 0; k2 < 4; ++k2) v[OFF + (k1 + 4 * k2) * STRIDE] = y[4 * k1 + k2];
    }
}

// ---- fused arithmetic ------------------------------------------------------------
//
// The transforms are bound by vector issue, so every butterfly (a + w b, a - w b) is written
// as six fused multiply-adds. A factor is kept as a scale and a ratio: with w = exp(-i t),
//     w b = cos t (b.x + tan t b.y,  b.y - tan t b.x)      (t up to pi/4, or any t: ratio = tan t)
//         = sin t (cot t b.x + b.y,  cot t b.y - b.x)      (t from pi/4 on: ratio = cot t),
// two multiply-adds for the pair in brackets, then one for each component of a + w b and a - w b,
// which are rounded independently of each other. (With w as it is, a + w b takes four and
// a - w b = 2a - (a + w b) two more, whose rounding adds to that of the sum: the transform of a
// padded row of 2048 is then off by 1.25e-7 of its norm, here by 1.11e-7, two-step 1.12e-7,
// evaluated on the CPU.)
// The bracket is at most |b| over the scale, so its rounding stays relative to |b| for
// any ratio. A radix-16 DFT by decimation in time takes its inputs' twiddles w^k along: level l
// multiplies by w^(8 >> l) W^c, so four levels of eight such butterflies (192 instructions) do
// the DFT and all fifteen input twiddles, against 160 + 60 for a 4 x 4 DFT after multiplying
// each input, and a thread holds 8 factors per pass instead of 15.

// Whether a transform is fused: below kFusedMin, where a call is bound by its launches, the
// two-step form is as fast and slightly more exact (a Fresnel plane of 128^2: 2.05e-7, fused
// 2.10e-7; of 256^2 2.46e-7 and 2.40e-7, of 2048^2 2.86e-7 and 2.65e-7).
constexpr bool fused_of(bool storage, int m) { return storage && m >= kFusedMin; }

// s = a + w b, b = a - w b, a = s with the factor (w.x, w.y): a factor that is not a table's.
__device__ __forceinline__ void bf_w(float2& a, float2& b, float wx, float wy) {
    const float sx = __fmaf_rn(-wy, b.y, __fmaf_rn(wx, b.x, a.x));
    const float sy = __fmaf_rn(wy, b.x, __fmaf_rn(wx, b.y, a.y));
    b = make_float2(__fmaf_rn(2.0f, a.x, -sx), __fmaf_rn(2.0f, a.y, -sy));
    a = make_float2(sx, sy);
}

// The same with the factor exp(-i t) as scale and ratio (sr.x, sr.y) for DIR = FWD, its
// conjugate for INV, times exp(DIR*i*pi/2) if ROT. COT: scale sin t and ratio cot t, else cos t
// and tan t.
template <int DIR, bool COT, bool ROT>
__device__ __forceinline__ void bf_sr(float2& a, float2& b, float2 sr) {
    constexpr float d = DIR == FWD ? 1.0f : -1.0f;
    float2 p = COT ? make_float2(__fmaf_rn(sr.y, b.x, d * b.y), __fmaf_rn(sr.y, b.y, -d * b.x))
                   : make_float2(__fmaf_rn(d * sr.y, b.y, b.x), __fmaf_rn(-d * sr.y, b.x, b.y));
    if constexpr (ROT) p = rot90<DIR>(p);
    b = make_float2(__fmaf_rn(-sr.x, p.x, a.x), __fmaf_rn(-sr.x, p.y, a.y));
    a = make_float2(__fmaf_rn(sr.x, p.x, a.x), __fmaf_rn(sr.x, p.y, a.y));
}

// Butterfly with the constant factor exp(DIR*2*pi*i*m/R), R <= 16.
template <int R, int M_, int DIR>
__device__ __forceinline__ void bf_const(float2& a, float2& b) {
    constexpr int m16 = M_ * (16 / R);  // angle in units of pi/8, 0..7
    static_assert(R <= 16 && m16 >= 0 && m16 < 8, "angle");
    if constexpr (m16 == 0 || m16 == 4) {
        const float2 t = m16 == 0 ? b : rot90<DIR>(b);
        b = csub(a, t);
        a = cadd(a, t);
    } else {
        constexpr bool cot = m16 == 3 || m16 == 5;
        constexpr double ctab[8] = {1.0, 0.92387953251128675613, 0.70710678118654752440,
                                    0.38268343236508977173, 0.0, -0.38268343236508977173,
                                    -0.70710678118654752440, -0.92387953251128675613};
        constexpr double c = cot ? ctab[m16 - 4 < 0 ? 4 - m16 : m16 - 4] : ctab[m16];  // the scale
        constexpr double s = cot ? ctab[m16] : ctab[m16 < 4 ? 4 - m16 : m16 - 4];
        constexpr float ratio = (float)(s / c);
        constexpr float scale = (float)((c + s * ratio) / (1.0 + (double)ratio * ratio));
        bf_sr<DIR, cot, false>(a, b, make_float2(scale, ratio));
    }
}

constexpr int bitrev(int v, int bits) {
    int r = 0;
    for (int i = 0; i < bits; ++i) r |= ((v >> i) & 1) << (bits - 1 - i);
    return r;
}

// One level of an untwisted radix-R decimation in time: pairs H = R >> (L+1) apart in each of
// 2^L groups, group g with the constant W_{2^(L+1)}^bitrev(g).
template <int R, int L, int DIR, int G>
__device__ __forceinline__ void dft_level_group(float2 (&u)[R]) {
    constexpr int H = R >> (L + 1);
#pragma unroll
    for (int k = 0; k < H; ++k) bf_const<(2 << L), bitrev(G, L), DIR>(u[G * 2 * H + k], u[G * 2 * H + H + k]);
}
template <int R, int L, int DIR>
__device__ __forceinline__ void dft_level(float2 (&u)[R]) {
    [&]<int... G>(std::integer_sequence<int, G...>) {
        (dft_level_group<R, L, DIR, G>(u), ...);
    }(std::make_integer_sequence<int, (1 << L)>{});
}
// Radix-R DFT from level L0 on (the levels before are the caller's); u[p] = X_bitrev(p).
template <int R, int DIR, int L0 = 0>
__device__ __forceinline__ void dft_const(float2 (&u)[R]) {
    if constexpr ((1 << L0) < R) {
        dft_level<R, L0, DIR>(u);
        dft_const<R, DIR, L0 + 1>(u);
    }
}

// Radix-16 DFT of u[k] w^k (w^-k for INV); u[p] = X_bitrev(p). t holds the table's factors
// w^8, w^4, w^2, w^2 W8, w, w W8, w W16, w W16^3 (those of an angle from pi/4 on, numbers 3, 5 and
// 7, with the ratio cot).
template <int DIR>
__device__ __forceinline__ void dft16_tw(float2 (&u)[16], const float2 (&t)[8]) {
#pragma unroll
    for (int k = 0; k < 8; ++k) bf_sr<DIR, false, false>(u[k], u[k + 8], t[0]);
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        bf_sr<DIR, false, false>(u[k], u[k + 4], t[1]);
        bf_sr<DIR, false, true>(u[k + 8], u[k + 12], t[1]);
    }
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        bf_sr<DIR, false, false>(u[k], u[k + 2], t[2]);
        bf_sr<DIR, false, true>(u[k + 4], u[k + 6], t[2]);
        bf_sr<DIR, true, false>(u[k + 8], u[k + 10], t[3]);
        bf_sr<DIR, true, true>(u[k + 12], u[k + 14], t[3]);
    }
    bf_sr<DIR, false, false>(u[0], u[1], t[4]);
    bf_sr<DIR, false, true>(u[2], u[3], t[4]);
    bf_sr<DIR, true, false>(u[4], u[5], t[5]);
    bf_sr<DIR, true, true>(u[6], u[7], t[5]);
    bf_sr<DIR, false, false>(u[8], u[9], t[6]);
    bf_sr<DIR, false, true>(u[10], u[11], t[6]);
    bf_sr<DIR, true, false>(u[12], u[13], t[7]);
    bf_sr<DIR, true, true>(u[14], u[15], t[7]);
}

// ---- pass plan and twiddles -----------------------------------------------------

constexpr int kE = 16;  // values per thread

template <int M>
struct Plan {
    static constexpr int LM = ilog2c(M);
    static constexpr int FIRST_BITS = (LM % 4) == 0 ? 4 : LM % 4;
    static constexpr int PASSES = 1 + (LM - FIRST_BITS) / 4;
    static constexpr int T = M / kE;
    static constexpr int R0 = 1 << FIRST_BITS;
    // product of the radices before pass p
    static constexpr int ns(int p) { return p == 0 ? 1 : R0 << (4 * (p - 1)); }
};

// The factors of every pass for one thread: held in registers from load() on, for the
// forward and the inverse transform, or (LAZY) read from the table before each pass, where the
// registers are wanted for other values (they are read before the exchange, while the
// transform's own values are in LDS).
template <int M, bool FUSED = fused_of(true, M), bool LAZY = false>
struct TwCache {
    using PL = Plan<M>;
    static constexpr int F = FUSED ? 8 : 16;  // factors per pass
    static constexpr int N = LAZY || PL::PASSES == 1 ? 1 : PL::PASSES - 1;
    float2 w[N][F];
    const float4* table;
    int j;
    template <int P>
    __device__ __forceinline__ void read(float2 (&x)[F]) const {
        constexpr int ns = PL::ns(P);
        int before = 0;
        for (int p = 1; p < P; ++p) before += PL::ns(p);
        const float4* t = table + before * (F / 2);
        const int k = j & (ns - 1);
#pragma unroll
        for (int q = 0; q < F / 2; ++q) {
            const float4 y = (t + q * ns)[k];
            x[2 * q] = make_float2(y.x, y.y);
            x[2 * q + 1] = make_float2(y.z, y.w);
        }
    }
    __device__ __forceinline__ void load_at(int jt, const float2* __restrict__ passes) {
        table = reinterpret_cast<const float4*>(passes);
        j = jt;
        if constexpr (!LAZY) {
            [&]<int... Ps>(std::integer_sequence<int, Ps...>) {
                (read<Ps + 1>(w[Ps]), ...);
            }(std::make_integer_sequence<int, PL::PASSES - 1>{});
        }
    }
    // tw: the table of length M
    __device__ __forceinline__ void load(int jt, const float2* __restrict__ tw) {
        load_at(jt, tw + (FUSED ? M : tw_at16(M)));
    }
    // twm: the table of length 2M
    __device__ __forceinline__ void load_half(int jt, const float2* __restrict__ twm) {
        load_at(jt, twm + (FUSED ? 2 * M : tw_at16(2 * M)) + F * tw_pass_k(2 * M));
    }
};

// ---- exchange through LDS -------------------------------------------------------
//
// C transforms are interleaved in one exchange area (element e of transform c at
// slot(e)*C + c); thread groups put the C transforms in consecutive lanes. Element e
// takes slot e + e/16: the strided Stockham writes then fall on different banks, and since
// no sum e0 + kk*Ns of a pass carries out of its low 4 bits, the 16 addresses of a
// pass differ by constants and cost no instructions.
__device__ __forceinline__ int lds_slot(int e) { return e + (e >> 4); }
constexpr int lds_off(int d) { return d + (d >> 4); }
template <int M>
constexpr int lds_elems() { return M + M / 16; }

// Block barrier for the LDS exchanges only. Threads of a block communicate through
// LDS alone (every global location is written by exactly one thread), so the
// barrier waits for this thread's LDS operations but leaves global loads and
// stores in flight; prefetched loads and the previous item's stores overlap the
// transform.
__device__ __forceinline__ void lds_barrier() {
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

// ---- transforms -------------------------------------------------------------------

// A pass leaves output out_of(p) of butterfly i at v[i*RP + p].
template <bool FUSED>
constexpr int out_of(int p, int bits) { return FUSED ? bitrev(p, bits) : p; }

// Outputs of pass P to LDS, then the inputs of the next pass back. Both barriers are
// block-wide.
template <int M, int P, int C, bool FUSED>
__device__ __forceinline__ void exchange(float2 (&v)[kE], float2* lds, int j, int c) {
    using PL = Plan<M>;
    constexpr int NS = PL::ns(P), RP = P == 0 ? PL::R0 : 16, T = PL::T, NB = kE / RP;
    constexpr int BITS = ilog2c(RP);
#pragma unroll
    for (int i = 0; i < NB; ++i) {
        const int e0 = P == 0 ? j * RP : (j / NS) * NS * 16 + (j & (NS - 1));
        float2* w = lds + lds_slot(e0) * C + c + (P == 0 ? lds_off(i * T * RP) * C : 0);
#pragma unroll
        for (int p = 0; p < RP; ++p) w[lds_off(out_of<FUSED>(p, BITS) * NS) * C] = v[i * RP + p];
    }
    lds_barrier();
    const float2* s = lds + lds_slot(j) * C + c;
#pragma unroll
    for (int r = 0; r < kE; ++r) v[r] = s[lds_off(r * T) * C];
    lds_barrier();
}

// The passes after the first: v holds the first pass's outputs; on exit v[r] = X[j + r*T].
template <int DIR, bool FUSED, int F>
__device__ __forceinline__ void pass16(float2 (&v)[kE], const float2 (&w)[F]) {
    if constexpr (FUSED) {
        dft16_tw<DIR>(v, w);
    } else {
#pragma unroll
        for (int k = 1; k < kE; ++k) v[k] = ctw<DIR>(v[k], w[k]);
        dft<16, DIR>(v);
    }
}
template <int M, int DIR, int C, int P, bool FUSED, bool LAZY>
__device__ __forceinline__ void later_passes(float2 (&v)[kE], float2* lds, int j, int c,
                                             const TwCache<M, FUSED, LAZY>& twc) {
    if constexpr (P < Plan<M>::PASSES) {
        if constexpr (LAZY) {
            float2 w[TwCache<M, FUSED, LAZY>::F];
            twc.template read<P>(w);
            exchange<M, P - 1, C, FUSED>(v, lds, j, c);
            pass16<DIR, FUSED>(v, w);
        } else {
            exchange<M, P - 1, C, FUSED>(v, lds, j, c);
            pass16<DIR, FUSED>(v, twc.w[P - 1]);
        }
        later_passes<M, DIR, C, P + 1>(v, lds, j, c, twc);
    } else {
        static_assert(M >= 16, "one radix-16 pass at least");
        float2 o[kE];
#pragma unroll
        for (int p = 0; p < kE; ++p) o[out_of<FUSED>(p, 4)] = v[p];
#pragma unroll
        for (int r = 0; r < kE; ++r) v[r] = o[r];
    }
}

// Transform of one sequence per thread group: on entry v[r] = x[j + r*T], on exit
// v[r] = X[j + r*T]. All threads of the block must call it (block barriers). lds: the
// exchange area of C interleaved transforms (C * lds_elems<M>() values), c < C this one's
// place. ZIN: x[M/2 ..] is zero and the registers of those elements are not read.
template <int M, int DIR, int C = 1, bool ZIN = false, bool FUSED, bool LAZY>
__device__ __forceinline__ void fft(float2 (&v)[kE], float2* lds, int j, int c,
                                    const TwCache<M, FUSED, LAZY>& twc) {
    constexpr int R0 = Plan<M>::R0, NB = kE / R0;
    float2 o[kE];
#pragma unroll
    for (int i = 0; i < NB; ++i) {
        float2 u[R0];
#pragma unroll
        for (int k = 0; k < R0; ++k) u[k] = v[i + (ZIN && k >= R0 / 2 ? k - R0 / 2 : k) * NB];
        if constexpr (!FUSED) dft<R0, DIR, 0, 1, ZIN>(u);
        else if constexpr (ZIN) dft_const<R0, DIR, 1>(u);  // level 0 of (x, 0): both outputs are x
        else dft_const<R0, DIR>(u);
#pragma unroll
        for (int k = 0; k < R0; ++k) o[i * R0 + k] = u[k];
    }
#pragma unroll
    for (int r = 0; r < kE; ++r) v[r] = o[r];
    later_passes<M, DIR, C, 1>(v, lds, j, c, twc);
}

// The same of the products x[j + r*T] h(r), h a per-element factor (the inverse transform
// after a transfer function). Fused: the first level's butterflies take the second factor of
// each pair as their own, which saves an addition per value. h(r) is called once for each r.
template <int M, int I, int K, class H>
__device__ __forceinline__ void mul_pair(const float2 (&v)[kE], H& h, float2 (&o)[kE]) {
    constexpr int R0 = Plan<M>::R0, NB = kE / R0, ra = I + K * NB, rb = ra + kE / 2;
    float2 p = cmul(v[ra], h(std::integral_constant<int, ra>{})), q = v[rb];
    const float2 g = h(std::integral_constant<int, rb>{});
    bf_w(p, q, g.x, g.y);
    o[I * R0 + K] = p;
    o[I * R0 + K + R0 / 2] = q;
}
template <int M, int DIR, int C, class H, bool FUSED, bool LAZY>
__device__ __forceinline__ void fft_mul(float2 (&v)[kE], H&& h, float2* lds, int j, int c,
                                        const TwCache<M, FUSED, LAZY>& twc) {
    if constexpr (!FUSED) {
        [&]<int... R>(std::integer_sequence<int, R...>) {
            ((v[R] = cmul(v[R], h(std::integral_constant<int, R>{}))), ...);
        }(std::make_integer_sequence<int, kE>{});
        fft<M, DIR, C>(v, lds, j, c, twc);
    } else {
        constexpr int R0 = Plan<M>::R0, NB = kE / R0;
        float2 o[kE];
        // pair n: butterfly n % NB, inputs n / NB and n / NB + R0/2
        [&]<int... N>(std::integer_sequence<int, N...>) {
            (mul_pair<M, N % NB, N / NB>(v, h, o), ...);
        }(std::make_integer_sequence<int, kE / 2>{});
#pragma unroll
        for (int i = 0; i < NB; ++i) {
            float2 u[R0];
#pragma unroll
            for (int k = 0; k < R0; ++k) u[k] = o[i * R0 + k];
            dft_const<R0, DIR, 1>(u);
#pragma unroll
            for (int k = 0; k < R0; ++k) o[i * R0 + k] = u[k];
        }
#pragma unroll
        for (int r = 0; r < kE; ++r) v[r] = o[r];
        later_passes<M, DIR, C, 1>(v, lds, j, c, twc);
    }
}

}  // namespace cwo
