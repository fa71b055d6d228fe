// Internal declarations shared by the HIP translation units of libeed4.
// Not part of the public ABI (include/eed4.h is).
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

namespace eed4 {

constexpr int kRMax = 8;        // largest Gaussian radius (sigma <= 8/3)
constexpr int kThreads = 256;   // threads per workgroup of the tile kernels

// Debug build (compiled with EED4_LDS_SENTINEL=1): every stencil kernel fills
// its LDS with NaN before each stage that writes it, so a read of a slot the
// stage did not write (an undersized halo, a missing barrier) turns the outputs
// it feeds into NaN or changes them.  Off (and compiled out) in the library.
#ifndef EED4_LDS_SENTINEL
#define EED4_LDS_SENTINEL 0
#endif
constexpr bool kLdsSentinel = EED4_LDS_SENTINEL != 0;

// NaN into p[0 .. n) by the whole workgroup, then a workgroup barrier.
__device__ __forceinline__ void sentinel_fill_block(float *p, int n)
{
    for (int i = threadIdx.x; i < n; i += blockDim.x) p[i] = __builtin_nanf("");
    __syncthreads();
}

// NaN into p[0 .. n) by one wave (its own LDS region); the wave's later LDS
// accesses stay after these stores.
__device__ __forceinline__ void sentinel_fill_wave(float *p, int n)
{
    for (int i = threadIdx.x & 63; i < n; i += 64) p[i] = __builtin_nanf("");
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront", "local");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront", "local");
}

// A kernel addresses the rows of a plane that one wave or workgroup touches with
// 32-bit byte offsets, which must stay below 2^31 (the offset of lanes without an
// output pixel): fewer than 256 rows at the largest width.  The most are the 170
// rows of a reverse strip of 136 output rows at R = 8; each geometry asserts it.
constexpr int kMaxWidth = 1 << 21;
constexpr bool rows_addressable(int rows) { return 4LL * kMaxWidth * rows < (1LL << 31); }

// Per-launch constants of one inner FSI step.
struct StepArgs {
    float w[2 * kRMax + 1];  // sampled Gaussian, w[j + R], j = -R..R, sums to 1
    float tau;               // time step
    float alpha;             // FSI weight alpha_k = (4k+2)/(2k+3)
    float inv_lam2;          // 1 / lambda^2
    int model;               // tensor variant: diffusivity | mu3 rule << 4 (0: FOEED)
};

// Tensor variants (the public flags EED4_DIFFUSIVITY / EED4_MU3).
constexpr int kNumDiffusivities = 4;   // Charbonnier, Perona-Malik, exp. Perona-Malik, Geman-Reynolds
constexpr int kNumMu3Rules = 3;        // geometric mean, arithmetic mean, maximum
constexpr int kDiffPeronaMalik = 1, kDiffPeronaMalikExp = 2, kDiffGemanReynolds = 3;
constexpr int kMu3Arithmetic = 1, kMu3Max = 2;
inline int model_of_flags(int flags) { return ((flags >> 16) & 0xf) | (((flags >> 20) & 0x3) << 4); }

// Workgroup tile of the fused step kernels: tw lanes (tw - 4 output columns)
// by th output rows.
struct TileShape {
    int tw, th;
};
constexpr int tile_cols(int tw) { return tw - 4; }

// Kernel shapes compiled into the library (index = config id): 0..2 and
// 9..10 are workgroup tiles (tw - 4 columns x th rows per 256 threads);
// 3..8 are wave strips: 3, 4, 7 and 8 of 124 columns (eed4_pair.h), 5 and 6 (and
// 3 on narrow images) of 60 (eed4_strip.h), by a segment of rows per wave.  The
// small tiles (9, 10) give images of a few hundred pixels a side more
// workgroups than the chip has CUs.
constexpr int kNumTileShapes = 5;
constexpr TileShape kTileShapes[kNumTileShapes] = {{64, 32}, {64, 16}, {32, 32}, {32, 16}, {16, 16}};
constexpr int kShapeStrip = 3;           // height by fit_strip_rows, or kShapeStripNarrow
constexpr int kShapeStripTall = 4;       // 136 rows
constexpr int kShapeStripShort = 5;      // >= 28 rows (more waves for small images)
constexpr int kShapeStripTiny = 6;       // >= 8 rows (shortest row pipeline per wave)
constexpr int kShapeStripWide = 7;       // 64 rows
constexpr int kShapeStripWideShort = 8;  // 28 rows
constexpr int kShapeTile32x16 = 9;
constexpr int kShapeTile16x16 = 10;
constexpr int kNumShapes = 11;
// What shape 3 runs where 60 columns fill the images' widths better than 124
// (fit_strip_shape): 60 columns x >= 64 rows.  Not a public id.
constexpr int kShapeStripNarrow = kNumShapes;
constexpr bool is_strip(int shape)
{
    return (shape >= kShapeStrip && shape <= kShapeStripWideShort) || shape == kShapeStripNarrow;
}
// index into kTileShapes of a tile shape
constexpr int tile_index(int shape) { return shape < kShapeStrip ? shape : shape - 6; }
constexpr bool is_pair(int shape)
{
    return is_strip(shape) && shape != kShapeStripShort && shape != kShapeStripTiny &&
           shape != kShapeStripNarrow;
}
constexpr int strip_width(int shape) { return is_pair(shape) ? 124 : 60; }

// Workgroups of `threads` threads one launch can have.  The runtime multiplies grid
// and block in 32 bits: it refuses 2^32 threads and silently runs the remainder
// beyond (2^24 + 1 workgroups of 256 run as one).
constexpr long long max_blocks(int threads) { return 0xffffffffLL / threads; }

// Launches over B images of `items` work items each, `per_block` items to a
// workgroup, in as few launches as max_blocks allows (one, short of millions of
// images): launch(b0, n, blocks) enqueues images b0 .. b0 + n - 1.
template <typename Launch>
hipError_t launch_batches(int B, long long items, int per_block, int threads, Launch &&launch)
{
    if (items <= 0 || B <= 0) return hipErrorInvalidValue;
    const long long most = max_blocks(threads) * per_block / items;    // images to a launch
    if (most < 1) return hipErrorInvalidValue;
    for (long long b0 = 0; b0 < B; b0 += most) {
        const int n = (int)(B - b0 < most ? B - b0 : most);
        launch((int)b0, n, (unsigned)((n * items + per_block - 1) / per_block));
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

// ---- launchers (eed4_forward.hip) ----
hipError_t launch_hold(float *u, const uint8_t *mask, const float *known, size_t n,
                       hipStream_t s);
hipError_t launch_step(int R, int shape, const float *ucur, const float *uprev, float *uout,
                       const float *ref, const uint8_t *mask, int B, int H, int W,
                       const StepArgs &a, double *partials, hipStream_t s);
// A step of the adjoint's forward recompute (the kernel follows the forward
// shape), which also writes K_sigma * u^k into vout.
hipError_t launch_step_keepv(int R, int shape, const float *ucur, const float *uprev,
                             float *uout, float *vout, const uint8_t *mask, int B, int H, int W,
                             const StepArgs &a, hipStream_t s);
// v = K_sigma * u, bitwise as a step from u computes it.
hipError_t launch_blur(int R, const float *u, float *v, int B, int H, int W, const StepArgs &a,
                       hipStream_t s);
hipError_t launch_reduce(const double *partials, int tiles_per_img, int B, double *sums,
                         hipStream_t s);
// residual partials per image of a launch over B images of H x W
int tiles_per_image(int shape, int R, int B, int H, int W);
int variant_shape(int R, int B, int H, int W);        // kernel shape of a tensor variant
// shape, or kShapeStripNarrow in the place of kShapeStrip, for B images of H[i] x W[i]
int fit_strip_shape(int shape, int B, const int *H, const int *W);
// output rows per strip segment in a launch over B images of the sizes
// (H[i], W[i]) with `copies` copies of each
int strip_rows(int R, int shape, int B, const int *H, const int *W, int copies);

}  // namespace eed4
