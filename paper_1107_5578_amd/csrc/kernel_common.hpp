// Configuration and helpers shared by the HIP kernel files of the diffraction path.
#pragma once
#include <cmath>
#include <cstdlib>
#include <cstddef>
#include <cstdint>
#include <map>
#include <mutex>
#include <type_traits>
#include <utility>

#include <hip/hip_ext.h>

#include "fft_device.hpp"
#include "launch.hpp"

namespace cwo {

// Every kernel of the library is launched through here: a plain launch, or with an armed
// stage timer one whose start and stop events the runtime stamps from the kernel's own
// execution (see StageTimer).
template <class K, class... A>
inline void launch_kernel(K kernel, dim3 grid, dim3 block, size_t shmem, hipStream_t s,
                          A... args) {
    if (StageTimer* t = g_stage_timer) {
        hipExtLaunchKernelGGL(kernel, grid, block, (std::uint32_t)shmem, s,
                              t->started ? nullptr : t->start, t->stop, 0u, args...);
        t->started = true;
    } else {
        hipLaunchKernelGGL(kernel, grid, block, shmem, s, args...);
    }
}

// ---- configuration per transform length --------------------------------------

// Row passes: one transform per thread group of T = M/E threads, RPB rows per block.
template <int M>
struct RowCfg {
    static constexpr int E = 16;
    static constexpr int T = M / E;
    static constexpr int RPB = (T >= 256) ? 1 : 256 / T;  // rows per block
    static constexpr int THREADS = T * RPB;
};

// ---- storage layout of the padded spectrum plane between the passes -------------
//
// Row-major: element (y, x) of the [Ny][Mx] plane at y*Mx + x. Tiled: the columns are
// grouped in tiles of kTileW and each tile stores its rows one after another, row y of tile t
// at place y ^ (m t mod Ny) of the tile: element (y, x) at
// (t*Ny + (y ^ (m t mod Ny)))*kTileW + x % kTileW, t = x / kTileW. In the tiled plane
// successive rows of a column lie kTileW values apart, so a wavefront of the column pass reads
// and writes a few whole cache lines instead of one line per lane, and a wavefront of a row
// pass moves the pieces of several rows in a tile together. Without the exclusive or, the
// pieces of one row would lie a power of two (Ny*32 bytes) apart, all on one channel of the
// caches and the memory; with it they are spread over all of them in runs of m rows. m = 32
// (1 KiB) for complex64; measured against m = 4 (one 128-byte line), 8, 16 and 64: one field
// of 512^2 17.3 us (m = 4: 18.3), of 1024^2 30.7 (32.7, 37.5, 36.5, 36.2), of 2048^2 87.7 (88,
// 94, 92, 87.5), of 4096^2 366 (364, 366, 419, 363), 8 fields of 1024^2 157 (181, 159, 157,
// 157). Planes of 16-bit storage keep m = 4: 2048^2 101 us (m = 32 105, 64 104).
//
// A thread addresses rows j + r*T (T a power of two, j < T) of its column as
// base + step(r*T) + lane: the lane part holds j, the step is uniform where t is.
constexpr int kTileW = 4;

struct LayRow {
    int mx;
    __device__ __forceinline__ unsigned lane(int j, int x, int, int) const { return (unsigned)j * mx + x; }
    __device__ __forceinline__ unsigned step(int rt, int, int) const { return (unsigned)rt * mx; }
};
template <class E>
struct LayTile {
    static constexpr unsigned kRun = sizeof(E) == 8 ? 32 : 4;  // m
    int ny;
    // place of row y in tile t
    __device__ __forceinline__ unsigned place(unsigned y, unsigned t) const { return y ^ ((kRun * t) & (ny - 1)); }
    __device__ __forceinline__ unsigned lane(int j, int x, int t, int T) const {
        return ((unsigned)t * ny + (place(j, t) & (T - 1))) * kTileW + (x % kTileW);
    }
    __device__ __forceinline__ unsigned step(int rt, int t, int T) const {
        return (place(rt, t) & ~(unsigned)(T - 1)) * kTileW;
    }
    // The same for one row y in the tiles tl + k*TS (TS a power of two, tl < TS): the first
    // element of the tile row is at tile_lane + tile_step(k*TS).
    __device__ __forceinline__ unsigned tile_lane(unsigned y, unsigned tl, unsigned TS) const {
        return (tl * ny + (place(y, tl) & (kRun * TS - 1))) * kTileW;
    }
    __device__ __forceinline__ size_t tile_step(unsigned y, unsigned kt, unsigned TS) const {
        return ((size_t)kt * ny + (place(y, kt) & ~(kRun * TS - 1))) * kTileW;
    }
};

// Row passes on the tiled plane: ROWS rows of one 128-byte line group per block in consecutive
// lanes, one row (16 values) per thread, so that the lanes of a wavefront hold ROWS*kTileW
// contiguous elements of each tile. (Two: with four, half as many blocks took 13.7 instead of
// 11.7 us for the 1024 rows of a 1024^2 field, and the 1024-thread blocks of 4096-point rows 26.5
// instead of 20.4.)
template <int M>
struct TileRowCfg {
    static constexpr int T = M / 16;
    static constexpr int ROWS = 2;
    static constexpr int THREADS = T * ROWS;
    static constexpr int LDS = ROWS * lds_elems<M>();  // float2
};

// Column pass: COLS adjacent columns per block in consecutive lanes, one column (16 values)
// per thread, so that a wavefront moves 8*COLS contiguous bytes per row and a thread with a
// fast transfer function keeps to 128 VGPRs: four waves per SIMD (see col_waves), where two
// columns and 30 twiddles per thread had two. Blocks are small (256 or 512 threads) so that
// several per CU are in different phases: at M = 4096 1024 threads (4 columns) took 58 us where 2
// columns take 44-48 and one 45; at M = 512 two columns (one wave per block) spread a 256^2 field
// over 256 blocks.
template <int M, int COLS_ = (M >= 2048 ? 2 : M >= 1024 ? 4 : M >= 512 ? 2 : 4096 / M)>
struct ColCfg {
    static constexpr int T = M / 16;
    static constexpr int COLS = COLS_;
    static constexpr int THREADS = T * COLS;
    static constexpr int LDS = COLS * lds_elems<M>();  // float2
    static constexpr int WAVES_PER_EU = 4;
};
// z-stack row inverse: its rows in the lanes of the column pass's columns (four lanes share a
// piece of a line: 366 us per 64 planes of 1024^2, with two 373, with eight 477).
template <int M>
using ZRowCfg = ColCfg<M, (M >= 4096 ? 2 : M >= 1024 ? 4 : M >= 512 ? 8 : 4096 / M)>;

// Column pass of the Fresnel Fourier form, on a row-major plane: wider pieces of a row (1024
// rows of 2048: 23.7 us for both passes with 8 columns, 24.4 with 4, 27.6 with 2).
template <int M>
using FfColCfg = ColCfg<M, (M >= 4096 ? 2 : M >= 2048 ? 4 : M >= 512 ? 8 : 4096 / M)>;

// z-stack column pass: the forward spectrum stays in registers while each plane's inverse
// transform runs on a copy. COLS columns in consecutive lanes, blocks of 128 threads where a
// column allows it (64 planes of 512^2: 82 us, with 256 threads 90; of 128^2 17 and 20).
template <int M>
struct ZColCfg {
    static constexpr int T = M / 16;
    static constexpr int COLS = T >= 256 ? 1 : T >= 64 ? 2 : T >= 8 ? 128 / T : 16;
    static constexpr int THREADS = T * COLS;
    static constexpr int LDS = COLS * lds_elems<M>();  // float2
};

// Consecutive workgroup ids are dispatched round-robin over the 8 XCDs, which
// have separate L2 caches. Remap so that each XCD works on a contiguous range
// of tiles; neighbouring tiles share cache lines.
__device__ __forceinline__ int xcd_remap(int bid, int nblocks) {
    if ((nblocks & 7) != 0) return bid;
    const int per = nblocks >> 3;
    return (bid & 7) * per + (bid >> 3);
}

// ---- host helpers -----------------------------------------------------------

#define CWO_DISPATCH_M(M_, ...)              \
    switch (M_) {                             \
        case 16: { constexpr int MM = 16; __VA_ARGS__; } break;     \
        case 32: { constexpr int MM = 32; __VA_ARGS__; } break;     \
        case 64: { constexpr int MM = 64; __VA_ARGS__; } break;     \
        case 128: { constexpr int MM = 128; __VA_ARGS__; } break;   \
        case 256: { constexpr int MM = 256; __VA_ARGS__; } break;   \
        case 512: { constexpr int MM = 512; __VA_ARGS__; } break;   \
        case 1024: { constexpr int MM = 1024; __VA_ARGS__; } break; \
        case 2048: { constexpr int MM = 2048; __VA_ARGS__; } break; \
        case 4096: { constexpr int MM = 4096; __VA_ARGS__; } break; \
        case 8192: { constexpr int MM = 8192; __VA_ARGS__; } break; \
        default: return hipErrorInvalidValue;                 \
    }

// Blocks of a persistent kernel that are resident at once on the current device (at
// most `items`). The occupancy query is answered once per kernel and device.
template <class K>
static int resident_blocks(K kernel, int threads, int items) {
    static std::mutex mu;
    static std::map<std::pair<const void*, int>, long long> cache;
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) dev = 0;
    const auto key = std::make_pair(reinterpret_cast<const void*>(kernel), dev);
    long long n = 0;
    {
        std::lock_guard<std::mutex> g(mu);
        auto it = cache.find(key);
        if (it != cache.end()) n = it->second;
    }
    if (n == 0) {
        int cus = 0, occ = 0;
        if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
            cus <= 0)
            cus = 256;
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&occ, kernel, threads, 0) != hipSuccess ||
            occ <= 0)
            occ = 1;
        n = (long long)occ * cus;
        std::lock_guard<std::mutex> g(mu);
        cache[key] = n;
    }
    return (int)(items < n ? items : n);
}

}  // namespace cwo
