// Forward kernels: Dirichlet hold, fused FSI inner step over a grid of
// tiles (one workgroup per tile, batch of equal-size images), and the
// deterministic FP64 reduction of the per-tile cycle residuals.
#include "eed4_internal.h"
#include "eed4_tile.h"
#include "eed4_pair.h"
#include "eed4_strip.h"

namespace eed4 {

// u = f on the known set K (eq. inpaintingModel).  Four pixels per thread,
// with the four mask bytes loaded (as one word when the mask is 4-byte
// aligned) before any of them is used, so the loads overlap.
__global__ __launch_bounds__(256) void hold_kernel(float *u, const uint8_t *__restrict__ mask,
                                                   const float *__restrict__ known, size_t n)
{
    const size_t i0 = ((size_t)blockIdx.x * blockDim.x + threadIdx.x) * 4;
    if (i0 >= n) return;
    unsigned m[4];
    if ((((uintptr_t)mask) & 3) == 0 && i0 + 4 <= n) {
        const unsigned wd = *reinterpret_cast<const unsigned *>(mask + i0);
#pragma unroll
        for (int j = 0; j < 4; ++j) m[j] = (wd >> (8 * j)) & 0xffu;
    } else {
#pragma unroll
        for (int j = 0; j < 4; ++j) m[j] = i0 + j < n ? mask[i0 + j] : 0u;
    }
#pragma unroll
    for (int j = 0; j < 4; ++j)
        if (m[j]) u[i0 + j] = known[i0 + j];
}

// Fused step over workgroup tiles.  RES adds the cycle residual, GEN selects the
// tensor variant at run time, VST also writes K_sigma * u^k (into vout).
template <int R, int TW, int TH, bool RES, bool GEN, bool VST>
__global__ __launch_bounds__(256) void step_kernel(
    const float *ucur, const float *uprev, float *uout, const float *ref,
    const uint8_t *__restrict__ mask, int H, int W, int nbx, int tiles_per_img, StepArgs a,
    double *partials, float *vout)
{
    __shared__ __attribute__((aligned(16))) float smem[TileGeo<R, TW, TH>::SMEM];
    const int tile = xcd_tile(blockIdx.x, gridDim.x);
    const int b = tile / tiles_per_img;
    const int t = tile - b * tiles_per_img;
    const int ty = t / nbx, tx = t - ty * nbx;
    const size_t off = (size_t)b * H * W;
    step_tile<R, TW, TH, kThreads, GEN, VST>(
        smem, ucur + off, uprev + off, uout + off, RES ? ref + off : nullptr, mask + off, H, W, ty,
        tx, a.w, a.tau, a.alpha, 0.25f * a.inv_lam2, RES ? partials + 2 * (size_t)tile : nullptr,
        a.model, VST ? vout + off : nullptr);
}

// The strip of a work item in the grid of strips and segments, as StripArgs.
__device__ __forceinline__ StripArgs strip_item(const float *ucur, const float *uprev, float *uout,
                                                const float *ref, float *vout, const uint8_t *mask,
                                                int H, int W, int nstrip, int per_img, int item,
                                                int sw, int oh, const StepArgs &a, int *seg_out)
{
    const int b = item / per_img;
    const int r = item - b * per_img;
    const int seg = r / nstrip, strip = r - seg * nstrip;
    const size_t off = (size_t)b * H * W;
    StripArgs s;
    s.ucur = ucur + off;
    s.uprev = uprev + off;
    s.uout = uout + off;
    s.ref = ref ? ref + off : nullptr;
    s.vout = vout ? vout + off : nullptr;
    s.mask = mask + off;
    s.H = H;
    s.W = W;
    s.X0 = strip * sw;
    s.Y0 = seg * oh;
    s.tau = a.tau;
    s.alpha = a.alpha;
    s.il2q = 0.25f * a.inv_lam2;
    s.model = a.model;
    s.up = 0;
    *seg_out = seg;
    return s;
}

// Fused step over 60-column wave strips.  GEN selects the tensor variant at run
// time (StepArgs::model); without it the kernel is the FOEED tensor.  VST also
// writes the presmoothed image K_sigma * u^k (into vout).
template <int R, bool RES, int ROWS, bool GEN, bool VST = false>
__device__ __forceinline__ void strip_kernel_body(const float *ucur, const float *uprev,
                                                  float *uout, const float *ref,
                                                  const uint8_t *__restrict__ mask, int H, int W,
                                                  int nstrip, int per_img, int nitems,
                                                  const StepArgs &a, double *partials,
                                                  float *vout = nullptr)
{
    using G = StripGeo<R, ROWS>;
    __shared__ float lds[4 * G::LDS];
    const int wave = threadIdx.x >> 6;
    // wave-uniform: keep the work item (and all that derives from it) in SGPRs
    const int item = __builtin_amdgcn_readfirstlane(xcd_tile(blockIdx.x, gridDim.x) * 4 + wave);
    if (item >= nitems) return;  // whole wave; the kernel has no workgroup barrier
    int seg;
    const StripArgs s = strip_item(ucur, uprev, uout, RES ? ref : nullptr, VST ? vout : nullptr,
                                   mask, H, W, nstrip, per_img, item, G::SW, G::OH, a, &seg);
    strip_step<R, RES, ROWS, GEN, VST>(lds + wave * G::LDS, s, a.w,
                                       RES ? partials + 2 * (size_t)item : nullptr);
}

template <int R, bool RES, int ROWS>
__global__ __launch_bounds__(256) void strip_kernel(const float *ucur, const float *uprev,
                                                    float *uout, const float *ref,
                                                    const uint8_t *__restrict__ mask, int H, int W,
                                                    int nstrip, int per_img, int nitems, StepArgs a,
                                                    double *partials)
{
    strip_kernel_body<R, RES, ROWS, false>(ucur, uprev, uout, ref, mask, H, W, nstrip, per_img,
                                           nitems, a, partials);
}

// Fused step over 124-column wave strips of `rows` rows (also VST: the step of
// the adjoint's recompute that keeps K_sigma * u^k).
template <int R, bool RES, bool VST>
__global__ __launch_bounds__(256) void pair_kernel(const float *ucur, const float *uprev,
                                                   float *uout, const float *ref, float *vout,
                                                   const uint8_t *__restrict__ mask, int H, int W,
                                                   int nstrip, int per_img, int nitems, int rows,
                                                   StepArgs a, double *partials)
{
    using G = PairGeo<R>;
    __shared__ __attribute__((aligned(16))) float lds[4 * G::LDS];
    const int wave = threadIdx.x >> 6;
    const int item = __builtin_amdgcn_readfirstlane(xcd_tile(blockIdx.x, gridDim.x) * 4 + wave);
    if (item >= nitems) return;
    int seg;
    StripArgs s = strip_item(ucur, uprev, uout, RES ? ref : nullptr, VST ? vout : nullptr, mask, H,
                             W, nstrip, per_img, item, G::SW, rows, a, &seg);
    s.up = seg & 1;
    pair_strip<R, RES, VST>(lds + wave * G::LDS, s, a.w, rows,
                            RES ? partials + 2 * (size_t)item : nullptr);
}

// The tensor variants (diffusivities of Table 7, mu3 choices of Sec. 3.1) on
// 60-column strips of >= 28 rows.
template <int R, bool RES>
__global__ __launch_bounds__(256) void strip_model_kernel(const float *ucur, const float *uprev,
                                                          float *uout, const float *ref,
                                                          const uint8_t *__restrict__ mask, int H,
                                                          int W, int nstrip, int per_img,
                                                          int nitems, StepArgs a, double *partials)
{
    strip_kernel_body<R, RES, 28, true>(ucur, uprev, uout, ref, mask, H, W, nstrip, per_img,
                                        nitems, a, partials);
}

// The step of the adjoint's forward recompute: u^{k+1} as strip_kernel (or
// strip_model_kernel when GEN) computes it, and K_sigma * u^k for the reverse
// step.
template <int R, int ROWS, bool GEN>
__global__ __launch_bounds__(256) void strip_keepv_kernel(const float *ucur, const float *uprev,
                                                          float *uout, float *vout,
                                                          const uint8_t *__restrict__ mask, int H,
                                                          int W, int nstrip, int per_img,
                                                          int nitems, StepArgs a)
{
    strip_kernel_body<R, false, ROWS, GEN, true>(ucur, uprev, uout, nullptr, mask, H, W, nstrip,
                                               per_img, nitems, a, nullptr, vout);
}

// v = K_sigma * u on the mirror-extended image (the presmoothing of Sec. 2.2)
// over 64 x 16 tiles with the fused step's stages A and B and its y pass, so v is
// bitwise the one a step from u computes.  (One LDS read per tap and pixel took
// 17.4 us on 2048^2 at R = 6, now 10.6.)  All 64 columns are outputs: no stencil
// follows that would take two of them on each side (64 x 2374x61 at R = 4 / 8:
// 30.5 / 40.5 us; with 60 output columns, two tiles across, 76.5 / 80).
constexpr int kBlurTW = 64, kBlurTH = 16;

// Geometry of a blur tile; the names are those of the step's tiles.
template <int R>
struct BlurGeo {
    static constexpr int OH = kBlurTH * kBlurTW / kThreads;   // output rows per wave
    static constexpr int h = R;                               // input halo
    static constexpr int SC = h;                              // staged columns left of the outputs
    static constexpr int OFF = SC - h;                        // first tap of lane 0's column
    static constexpr int UH = kBlurTH + 2 * h;                // staged rows
    static constexpr int UQ = (SC + kBlurTW + h + 3) / 4;     // 16-byte loads per staged row
    static constexpr int NF4 = (OFF + 4 + 2 * R + 3) / 4;     // 16-byte LDS reads per x-pass item
    static constexpr int NQ = kBlurTW / 4;                    // x-pass items per row
    static constexpr int UW = 4 * (UQ > NF4 + NQ - 1 ? UQ : NF4 + NQ - 1);   // row stride of u
    static constexpr int NA = UH * UQ, NB = UH * NQ;          // items of stages A and B
    static constexpr int NU = UH * UW, NX = UH * kBlurTW;
    static constexpr int SMEM = NU + NX;                      // floats of LDS
    static constexpr int IA = (NA + kThreads - 1) / kThreads; // stage A items per thread
    static_assert(rows_addressable(UH), "row offsets");
};

template <int R>
__global__ __launch_bounds__(256) void blur_kernel(const float *u_all, float *v_all, int H, int W,
                                                   int nbx, int tiles_per_img, StepArgs a)
{
    using G = BlurGeo<R>;
    __shared__ __attribute__((aligned(16))) float smem[G::SMEM];
    float *sU = smem, *sX = smem + G::NU;
    const int tile = __builtin_amdgcn_readfirstlane(xcd_tile(blockIdx.x, gridDim.x));
    const int b = tile / tiles_per_img;
    const int t = tile - b * tiles_per_img;
    const int Y0 = (t / nbx) * kBlurTH, X0 = (t - (t / nbx) * nbx) * kBlurTW;
    const int lane = threadIdx.x & 63;
    const int grp = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), Yg = Y0 + grp * G::OH;
    if constexpr (kLdsSentinel) sentinel_fill_block(smem, G::SMEM);
    const unsigned W4 = 4u * (unsigned)W;
    const int y0 = Y0 - G::h, b0 = y0 > 0 ? y0 : 0;
    const int nb = H - b0 < G::UH ? H - b0 : G::UH;
    const size_t base = (size_t)b * H * W + (size_t)b0 * W;
    const __amdgpu_buffer_rsrc_t rs_u = buffer_rsrc(u_all + base, (unsigned)nb * W4);
    const __amdgpu_buffer_rsrc_t rs_v = buffer_rsrc(v_all + base, (unsigned)nb * W4);
    f32x4 st[G::IA];
    tile_load<G, kThreads>(st, rs_u, X0 - G::SC, y0, b0, H, W);
    tile_put<G, kThreads>(sU, st);
    float wv[2 * R + 1];
    vector_weights<R>(a.w, wv);
    __syncthreads();
    tile_xpass<R, kBlurTW, G, kThreads>(sU, sX, wv);
    __syncthreads();
    const int c = X0 + lane;
    const unsigned vo = c < W ? 4u * (unsigned)c : kOffNone;
    const float *px = sX + 64 * (grp * G::OH) + lane;                // row Yg - R
#pragma unroll
    for (int j = 0; j < G::OH; ++j) {
        const float x = ypass_sym<R>(wv, [&](int t) { return px[64 * (j + R + t)]; });
        if (Yg + j < H)
            __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(x), rs_v, vo,
                                                  uniform_row(Yg + j - b0) * W4, 0);
    }
}

// sums[b] = fixed-order sum of the residual partials of image b's tiles.
__global__ __launch_bounds__(1024) void reduce_kernel(const double *partials, int tiles_per_img,
                                                      double *sums)
{
    __shared__ double sd[1024], sn[1024];
    const int b = blockIdx.x;
    const double *p = partials + 2 * (size_t)b * tiles_per_img;
    double d = 0.0, n = 0.0;
#pragma unroll 4
    for (int i = threadIdx.x; i < tiles_per_img; i += 1024) {
        d += p[2 * i];
        n += p[2 * i + 1];
    }
    sd[threadIdx.x] = d;
    sn[threadIdx.x] = n;
    __syncthreads();
    for (int s = 512; s > 0; s >>= 1) {
        if (threadIdx.x < s) {
            sd[threadIdx.x] += sd[threadIdx.x + s];
            sn[threadIdx.x] += sn[threadIdx.x + s];
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        sums[2 * b] = sd[0];
        sums[2 * b + 1] = sn[0];
    }
}

hipError_t launch_hold(float *u, const uint8_t *mask, const float *known, size_t n,
                       hipStream_t s)
{
    constexpr size_t kPart = (size_t)1 << 33;     // elements to a launch: 2^23 workgroups
    for (size_t i = 0; i < n; i += kPart) {
        const size_t m = n - i < kPart ? n - i : kPart;
        hipLaunchKernelGGL(hold_kernel, dim3((unsigned)((m + 1023) / 1024)), dim3(256), 0, s, u + i,
                           mask + i, known + i, m);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

// Segment height of the default 124-column strips in a launch of `waves(rows)`
// waves.  A wave's time is proportional to the rows it streams (the outputs,
// four more, and the prologue, of which a row costs about half) and, per row,
// measured on full launches of 1, 2, 3 and 4 waves a SIMD (4096^2 and 2900^2,
// R = 5 and 6): 0.475, 0.6, 0.8 and 1.03 us.  Three waves fit a SIMD's
// registers from R = 6 on, four below.  So a launch that leaves a few waves for
// another round on the SIMDs costs a whole round: 4096^2 at R = 6 takes 47.9 us
// with 48 rows (2924 waves for 3072 places), 52.3 us with 36 (3876), 54.6 with
// 64 (2176).
template <typename Waves>
static int fit_strip_rows(int R, Waves &&waves)
{
    constexpr double kRowTime[5] = {0.0, 0.475, 0.6, 0.8, 1.03};
    constexpr long long kSimds = 1024;
    const long long fit = R <= 5 ? 4 : 3;
    int best = 0;
    double best_cost = 0.0;
    for (int rows = 28; rows <= 136; rows += 4) {
        const long long n = (waves(rows) + kSimds - 1) / kSimds;      // waves per SIMD
        const double cost = ((double)(n / fit) * kRowTime[fit] + kRowTime[n % fit]) * (rows + R + 6);
        if (best == 0 || cost < best_cost) {
            best = rows;
            best_cost = cost;
        }
    }
    return best;
}

int strip_rows(int R, int shape, int B, const int *H, const int *W, int copies)
{
    switch (shape) {
    case kShapeStripTall: return 136;
    case kShapeStripWide: return 64;
    case kShapeStripWideShort: return 28;
    case kShapeStrip:
        return fit_strip_rows(R, [&](int rows) {
            long long n = 0;
            for (int i = 0; i < B; ++i)
                n += (long long)((W[i] + 123) / 124) * ((H[i] + rows - 1) / rows);
            return n * copies;
        });
    default: break;
    }
    switch (R) {
#define EED4_CASE(r) \
    case r: return shape == kShapeStripNarrow  ? StripGeo<r, 64>::OH \
                   : shape == kShapeStripShort ? StripGeo<r, 28>::OH \
                                               : StripGeo<r, 8>::OH;
        EED4_CASE(0) EED4_CASE(1) EED4_CASE(2) EED4_CASE(3) EED4_CASE(4)
        EED4_CASE(5) EED4_CASE(6) EED4_CASE(7) EED4_CASE(8)
#undef EED4_CASE
    default: return 0;
    }
}

// Shape 3 runs strips of 124 columns unless those of 60, whose lanes each take one
// column, cover the images' widths with a sixth fewer columns in all, or the images
// are at most 64 wide (one wave of 124 columns would be half empty, and all of it at
// the border).  R = 3 / R = 8, us a step, 124 columns against 60: 500 x 128^2 35.7
// and 29.8 / 46.2 and 36.6, 131072x130 37.7 and 28.7 / 45.8 and 37.9, 40000x250 33.6
// and 29.7 / 44.1 and 42.1, 4000 x 48^2 46.9 and 28.3 / 66.9 and 42.4, 2000 x 64^2 37.3
// and 34.8 / 46.6 and 43.4.  Where the 60 columns save less they are mostly slower:
// 16000x380 (15 % fewer) 23.1 and 23.5 / 29.6 and 29.7, 2300x2900 20.3 and 23.5 / 28.1
// and 29.7, 4096^2 40.6 and 42.1 / 51.7 and 53.5.
int fit_strip_shape(int shape, int B, const int *H, const int *W)
{
    if (shape != kShapeStrip) return shape;
    double narrow = 0.0, wide = 0.0;                      // columns covered, times rows
    for (int i = 0; i < B; ++i) {
        narrow += (W[i] <= 64 ? 1.0 : 1.2) * H[i] * ((W[i] + 59) / 60 * 60);
        wide += (double)H[i] * ((W[i] + 123) / 124 * 124);
    }
    return narrow <= wide ? kShapeStripNarrow : shape;
}

int tiles_per_image(int shape, int R, int B, int H, int W)
{
    shape = fit_strip_shape(shape, 1, &H, &W);
    if (is_strip(shape)) {
        const int oh = strip_rows(R, shape, 1, &H, &W, B), sw = strip_width(shape);
        if (oh <= 0) return 0;
        return ((W + sw - 1) / sw) * ((H + oh - 1) / oh);
    }
    const TileShape ts = kTileShapes[tile_index(shape)];
    const int sw = tile_cols(ts.tw);
    return ((W + sw - 1) / sw) * ((H + ts.th - 1) / ts.th);
}

// Kernel shape a tensor variant runs (the public shape id of a variant stays
// kShapeStripShort): the strips from about 3072 waves on, where they are level
// with the 60 x 32 tiles (FOEED at 2560^2: 25.5 against 25.8 us; the variants
// at 2048^2 24.6 against 19.2 us, at 2896^2 30.4 against 32.1 us), and 60 x 16
// tiles where those of 32 rows would be fewer than four a CU (1024^2: 8.6 us,
// 28-row strips 20.6 us).
int variant_shape(int R, int B, int H, int W)
{
    const long long waves = (long long)tiles_per_image(kShapeStripShort, R, B, H, W) * B;
    if (waves >= 3072) return kShapeStripShort;
    return (long long)tiles_per_image(0, R, B, H, W) * B >= 1024 ? 0 : 1;
}

template <int R, int ROWS, bool GEN = false>
static hipError_t launch_strip_t(const float *ucur, const float *uprev, float *uout,
                                 const float *ref, const uint8_t *mask, int B, int H, int W,
                                 const StepArgs &a, double *partials, hipStream_t s)
{
    using G = StripGeo<R, ROWS>;
    const int nstrip = (W + G::SW - 1) / G::SW;
    const int per_img = nstrip * ((H + G::OH - 1) / G::OH);
    static_assert(!GEN || ROWS == 28, "tensor variants run 28-row strips");
    return launch_batches(B, per_img, 4, 256, [&](int b0, int n, unsigned blocks) {
        const size_t o = (size_t)b0 * H * W;
        const float *r = ref ? ref + o : nullptr;
        double *const pt = ref ? partials + 2 * (size_t)b0 * per_img : nullptr;
        const dim3 g(blocks), b(256);
        if constexpr (GEN) {
            if (ref)
                hipLaunchKernelGGL((strip_model_kernel<R, true>), g, b, 0, s, ucur + o, uprev + o,
                                   uout + o, r, mask + o, H, W, nstrip, per_img, per_img * n, a, pt);
            else
                hipLaunchKernelGGL((strip_model_kernel<R, false>), g, b, 0, s, ucur + o, uprev + o,
                                   uout + o, r, mask + o, H, W, nstrip, per_img, per_img * n, a, pt);
        } else if (ref) {
            hipLaunchKernelGGL((strip_kernel<R, true, ROWS>), g, b, 0, s, ucur + o, uprev + o,
                               uout + o, r, mask + o, H, W, nstrip, per_img, per_img * n, a, pt);
        } else {
            hipLaunchKernelGGL((strip_kernel<R, false, ROWS>), g, b, 0, s, ucur + o, uprev + o,
                               uout + o, r, mask + o, H, W, nstrip, per_img, per_img * n, a, pt);
        }
    });
}

// A pair shape; with vout the recompute step that keeps K_sigma * u^k.
template <int R>
static hipError_t launch_pair_r(int shape, const float *ucur, const float *uprev, float *uout,
                                const float *ref, float *vout, const uint8_t *mask, int B, int H,
                                int W, const StepArgs &a, double *partials, hipStream_t s)
{
    const int rows = strip_rows(R, shape, 1, &H, &W, B);
    const int nstrip = (W + PairGeo<R>::SW - 1) / PairGeo<R>::SW;
    const int per_img = nstrip * ((H + rows - 1) / rows);
    return launch_batches(B, per_img, 4, 256, [&](int b0, int n, unsigned blocks) {
        const size_t o = (size_t)b0 * H * W;
        const dim3 g(blocks), b(256);
        if (vout)
            hipLaunchKernelGGL((pair_kernel<R, false, true>), g, b, 0, s, ucur + o, uprev + o,
                               uout + o, nullptr, vout + o, mask + o, H, W, nstrip, per_img,
                               per_img * n, rows, a, nullptr);
        else if (ref)
            hipLaunchKernelGGL((pair_kernel<R, true, false>), g, b, 0, s, ucur + o, uprev + o,
                               uout + o, ref + o, nullptr, mask + o, H, W, nstrip, per_img,
                               per_img * n, rows, a, partials + 2 * (size_t)b0 * per_img);
        else
            hipLaunchKernelGGL((pair_kernel<R, false, false>), g, b, 0, s, ucur + o, uprev + o,
                               uout + o, nullptr, nullptr, mask + o, H, W, nstrip, per_img,
                               per_img * n, rows, a, nullptr);
    });
}

template <int R, int ROWS, bool GEN>
static hipError_t launch_keepv_t(const float *ucur, const float *uprev, float *uout, float *vout,
                                 const uint8_t *mask, int B, int H, int W, const StepArgs &a,
                                 hipStream_t s)
{
    using G = StripGeo<R, ROWS>;
    const int nstrip = (W + G::SW - 1) / G::SW;
    const int per_img = nstrip * ((H + G::OH - 1) / G::OH);
    return launch_batches(B, per_img, 4, 256, [&](int b0, int n, unsigned blocks) {
        const size_t o = (size_t)b0 * H * W;
        hipLaunchKernelGGL((strip_keepv_kernel<R, ROWS, GEN>), dim3(blocks), dim3(256), 0, s, ucur + o,
                           uprev + o, uout + o, vout + o, mask + o, H, W, nstrip, per_img,
                           per_img * n, a);
    });
}

template <int R>
static hipError_t launch_blur_r(const float *u, float *v, int B, int H, int W, const StepArgs &a,
                                hipStream_t s)
{
    const int nbx = (W + kBlurTW - 1) / kBlurTW, nby = (H + kBlurTH - 1) / kBlurTH;
    return launch_batches(B, (long long)nbx * nby, 1, 256, [&](int b0, int, unsigned blocks) {
        const size_t o = (size_t)b0 * H * W;
        hipLaunchKernelGGL((blur_kernel<R>), dim3(blocks), dim3(256), 0, s, u + o, v + o, H, W, nbx,
                           nbx * nby, a);
    });
}

template <int R, int TW, int TH, bool GEN = false>
static hipError_t launch_step_t(const float *ucur, const float *uprev, float *uout,
                                const float *ref, const uint8_t *mask, int B, int H, int W,
                                const StepArgs &a, double *partials, hipStream_t s)
{
    const int nbx = (W + tile_cols(TW) - 1) / tile_cols(TW), nby = (H + TH - 1) / TH;
    const int tpi = nbx * nby;
    return launch_batches(B, tpi, 1, 256, [&](int b0, int, unsigned blocks) {
        const size_t o = (size_t)b0 * H * W;
        const dim3 g(blocks), b(256);
        if (ref)
            hipLaunchKernelGGL((step_kernel<R, TW, TH, true, GEN, false>), g, b, 0, s, ucur + o,
                               uprev + o, uout + o, ref + o, mask + o, H, W, nbx, tpi, a,
                               partials + 2 * (size_t)b0 * tpi, nullptr);
        else
            hipLaunchKernelGGL((step_kernel<R, TW, TH, false, GEN, false>), g, b, 0, s, ucur + o,
                               uprev + o, uout + o, nullptr, mask + o, H, W, nbx, tpi, a, nullptr,
                               nullptr);
    });
}

template <int R, int TW, int TH, bool GEN>
static hipError_t launch_keepv_tile(const float *ucur, const float *uprev, float *uout, float *vout,
                                    const uint8_t *mask, int B, int H, int W, const StepArgs &a,
                                    hipStream_t s)
{
    const int nbx = (W + tile_cols(TW) - 1) / tile_cols(TW), nby = (H + TH - 1) / TH;
    return launch_batches(B, (long long)nbx * nby, 1, 256, [&](int b0, int, unsigned blocks) {
        const size_t o = (size_t)b0 * H * W;
        hipLaunchKernelGGL((step_kernel<R, TW, TH, false, GEN, true>), dim3(blocks), dim3(256), 0, s,
                           ucur + o, uprev + o, uout + o, nullptr, mask + o, H, W, nbx, nbx * nby, a,
                           nullptr, vout + o);
    });
}

template <int R>
static hipError_t launch_step_r(int shape, const float *ucur, const float *uprev, float *uout,
                                const float *ref, const uint8_t *mask, int B, int H, int W,
                                const StepArgs &a, double *partials, hipStream_t s)
{
    if (a.model != 0) {              // tensor variants: the shapes of variant_shape
        switch (shape) {
        case 0: return launch_step_t<R, 64, 32, true>(ucur, uprev, uout, ref, mask, B, H, W, a, partials, s);
        case 1: return launch_step_t<R, 64, 16, true>(ucur, uprev, uout, ref, mask, B, H, W, a, partials, s);
        case kShapeStripShort: return launch_strip_t<R, 28, true>(ucur, uprev, uout, ref, mask, B, H, W, a, partials, s);
        default: return hipErrorInvalidValue;
        }
    }
    switch (shape) {
    case 0: return launch_step_t<R, 64, 32>(ucur, uprev, uout, ref, mask, B, H, W, a, partials, s);
    case 1: return launch_step_t<R, 64, 16>(ucur, uprev, uout, ref, mask, B, H, W, a, partials, s);
    case 2: return launch_step_t<R, 32, 32>(ucur, uprev, uout, ref, mask, B, H, W, a, partials, s);
    case kShapeStripShort: return launch_strip_t<R, 28>(ucur, uprev, uout, ref, mask, B, H, W, a, partials, s);
    case kShapeStripTiny: return launch_strip_t<R, 8>(ucur, uprev, uout, ref, mask, B, H, W, a, partials, s);
    case kShapeStripNarrow: return launch_strip_t<R, 64>(ucur, uprev, uout, ref, mask, B, H, W, a, partials, s);
    case kShapeStrip: case kShapeStripTall: case kShapeStripWide: case kShapeStripWideShort:
        return launch_pair_r<R>(shape, ucur, uprev, uout, ref, nullptr, mask, B, H, W, a, partials, s);
    case kShapeTile32x16: return launch_step_t<R, 32, 16>(ucur, uprev, uout, ref, mask, B, H, W, a, partials, s);
    case kShapeTile16x16: return launch_step_t<R, 16, 16>(ucur, uprev, uout, ref, mask, B, H, W, a, partials, s);
    default: return hipErrorInvalidValue;
    }
}

// The keep-v step of a forward step shape: a strip shape keeps its own (8-row
// strips aside); of the 60-column tiles those of 32 rows, which recompute fewer
// halo rows, run from more than two a CU on (beside the reverse step the sum of
// the work counts: 16 x 256^2 at R = 3, backward of 50 steps 893 us against 925
// with 16 rows; 1000^2 872 and 880), those of 16 rows below (700^2 702 against
// 708, 64 x 100^2 734 against 741).
template <int R, bool GEN>
static hipError_t launch_keepv_r(int shape, const float *ucur, const float *uprev, float *uout,
                                 float *vout, const uint8_t *mask, int B, int H, int W,
                                 const StepArgs &a, hipStream_t s)
{
    switch (shape) {
    case 0: return launch_keepv_tile<R, 64, 32, GEN>(ucur, uprev, uout, vout, mask, B, H, W, a, s);
    case kShapeStripShort:
        return launch_keepv_t<R, 28, GEN>(ucur, uprev, uout, vout, mask, B, H, W, a, s);
    case kShapeStripNarrow:
        if constexpr (!GEN)
            return launch_keepv_t<R, 64, false>(ucur, uprev, uout, vout, mask, B, H, W, a, s);
        return hipErrorInvalidValue;
    case kShapeStrip: case kShapeStripTall: case kShapeStripWide: case kShapeStripWideShort:
        if constexpr (!GEN)
            return launch_pair_r<R>(shape, ucur, uprev, uout, nullptr, vout, mask, B, H, W, a,
                                    nullptr, s);
        return hipErrorInvalidValue;
    default:
        if ((long long)tiles_per_image(0, R, B, H, W) * B > 512)
            return launch_keepv_tile<R, 64, 32, GEN>(ucur, uprev, uout, vout, mask, B, H, W, a, s);
        return launch_keepv_tile<R, 64, 16, GEN>(ucur, uprev, uout, vout, mask, B, H, W, a, s);
    }
}

hipError_t launch_step(int R, int shape, const float *ucur, const float *uprev, float *uout,
                       const float *ref, const uint8_t *mask, int B, int H, int W,
                       const StepArgs &a, double *partials, hipStream_t s)
{
    shape = fit_strip_shape(shape, 1, &H, &W);
    switch (R) {
#define EED4_CASE(r) \
    case r: return launch_step_r<r>(shape, ucur, uprev, uout, ref, mask, B, H, W, a, partials, s);
        EED4_CASE(0) EED4_CASE(1) EED4_CASE(2) EED4_CASE(3) EED4_CASE(4)
        EED4_CASE(5) EED4_CASE(6) EED4_CASE(7) EED4_CASE(8)
#undef EED4_CASE
    default: return hipErrorInvalidValue;
    }
}

hipError_t launch_step_keepv(int R, int shape, const float *ucur, const float *uprev,
                             float *uout, float *vout, const uint8_t *mask, int B, int H, int W,
                             const StepArgs &a, hipStream_t s)
{
    shape = fit_strip_shape(shape, 1, &H, &W);
    switch (R) {
#define EED4_CASE(r) \
    case r:                                                                                   \
        return a.model != 0                                                                   \
                   ? launch_keepv_r<r, true>(shape, ucur, uprev, uout, vout, mask, B, H, W, a, s) \
                   : launch_keepv_r<r, false>(shape, ucur, uprev, uout, vout, mask, B, H, W, a, s);
        EED4_CASE(0) EED4_CASE(1) EED4_CASE(2) EED4_CASE(3) EED4_CASE(4)
        EED4_CASE(5) EED4_CASE(6) EED4_CASE(7) EED4_CASE(8)
#undef EED4_CASE
    default: return hipErrorInvalidValue;
    }
}

hipError_t launch_blur(int R, const float *u, float *v, int B, int H, int W, const StepArgs &a,
                       hipStream_t s)
{
    switch (R) {
#define EED4_CASE(r) case r: return launch_blur_r<r>(u, v, B, H, W, a, s);
        EED4_CASE(0) EED4_CASE(1) EED4_CASE(2) EED4_CASE(3) EED4_CASE(4)
        EED4_CASE(5) EED4_CASE(6) EED4_CASE(7) EED4_CASE(8)
#undef EED4_CASE
    default: return hipErrorInvalidValue;
    }
}

hipError_t launch_reduce(const double *partials, int tiles_per_img, int B, double *sums,
                         hipStream_t s)
{
    return launch_batches(B, 1, 1, 1024, [&](int b0, int, unsigned blocks) {
        hipLaunchKernelGGL(reduce_kernel, dim3(blocks), dim3(1024), 0, s,
                           partials + 2 * (size_t)b0 * tiles_per_img, tiles_per_img, sums + 2 * (size_t)b0);
    });
}

}  // namespace eed4
