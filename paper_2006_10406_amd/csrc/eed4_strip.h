// Device code of one fused FOEED/FSI inner step on a vertical strip, one
// wavefront per strip, no workgroup barriers (the short segments, images whose
// width 60 columns fill better than 124, and the tensor variants; eed4_pair.h has
// the wide and tall ones).
//
// A wave owns 64 consecutive columns c = X0-2 .. X0+61, one per lane, and
// streams down the rows of a segment.  For each input row y it
//   S1  stages u^k(y, X0-2-R .. X0+61+R) in a per-wave LDS ring (mirrored
//       indices realise the Neumann condition, Sec. 2.1) and takes the x pass
//       of the Gaussian presmoothing (Sec. 2.2) at its columns;
//   S2  completes the y pass at row y-R from a register window of the last
//       2R+1 x-pass values (the row loop is unrolled over that window);
//   S3  at row g = y-R-1: central-difference gradient of u_sigma, fourth-order
//       diffusion tensor (Sec. 3.1: eigenvalues g, 1, sqrt g), Hessian of u
//       from the LDS ring (Sec. 3.3 stencils, sign-corrected u_xy) and
//       T = D : H;
//   S4  at row o = g-1: outer differences of T (eq. genModel), explicit step,
//       FSI extrapolation (Sec. 3.3), Dirichlet hold; optional FP64 residual;
//       optionally also the presmoothed image v = K_sigma * u^k at row o (the
//       adjoint's recompute keeps it for the reverse step).
// Horizontal neighbours across lanes come from DPP wave shifts.  Outputs are
// the 60 columns X0 .. X0+59.  Every intermediate lives on the mirror-extended
// image, so P stays symmetric.
#pragma once

#include "eed4_internal.h"
#include "eed4_pointwise.h"

namespace eed4 {

// Half-sample mirror by repeated reflection (any i, n >= 1).
__device__ __forceinline__ int mirror_reflect(int i, int n)
{
    while (i < 0 || i >= n) i = (i < 0) ? -1 - i : 2 * n - 1 - i;
    return i;
}

// Value held by lane+1 / lane-1 (DPP wave shifts; edge lanes read 0).
__device__ __forceinline__ float from_next_lane(float v)
{
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x130, 0xF, 0xF, true));
}
__device__ __forceinline__ float from_prev_lane(float v)
{
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x138, 0xF, 0xF, true));
}

// Lane 0's value of a double, wave-uniform.
__device__ __forceinline__ double lane0_double(double x)
{
    const unsigned long long b = (unsigned long long)__double_as_longlong(x);
    const unsigned lo = __builtin_amdgcn_readlane((unsigned)b, 0);
    const unsigned hi = __builtin_amdgcn_readlane((unsigned)(b >> 32), 0);
    return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}

// Orders LDS accesses of different lanes of one wave (a wave executes its LDS
// instructions in order; this only stops the compiler from reordering them).
__device__ __forceinline__ void wave_lds_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront", "local");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront", "local");
}

// ROWS is the least number of output rows of a wave's segment (the segment
// is rounded up to whole unrolled iterations).
//
// The LDS ring holds the last D staged rows column-major: staged column c
// (0 .. NU-1) of ring row r is at (c + 1) * CS + r, with an empty column on
// each side.  A lane addresses everything it reads (x-pass taps, Hessian
// neighbours) as compile-time offsets from its own column, which stay within
// the reach of paired LDS reads, and the odd stride CS keeps the 64 lanes on
// distinct banks.
template <int R, int ROWS>
struct StripGeo {
    static constexpr int P = 2 * R + 1;                       // y window length
    static constexpr int U = P * ((R + 3 + P - 1) / P);       // unroll = LDS ring depth
    static constexpr int D = U;                               // (a multiple of P, >= R+3)
    static constexpr int h = R + 2;                           // input halo
    static constexpr int SW = 60;                             // output columns per wave
    static constexpr int NU = 64 + 2 * R;                     // staged u columns per row
    static constexpr int CS = D | 1;                          // ring column stride (odd)
    static constexpr int M = (ROWS + 4 + U - 1) / U;          // main-loop iterations
    static constexpr int NROW = 2 * R + M * U;                // rows streamed per wave
    static constexpr int OH = NROW - 2 * h;                   // output rows per wave
    static constexpr int LDS = (NU + 2) * CS;                 // floats of LDS per wave
    static_assert(rows_addressable(NROW), "row offsets");
};

// Per-wave constants of a strip step.
struct StripArgs {
    const float *ucur, *uprev;
    float *uout;
    const float *ref;           // cycle start for the residual (RES variant only)
    float *vout;                // K_sigma * u^k at the output pixels (VST variant only)
    const uint8_t *mask;
    int H, W, X0, Y0;
    float tau, alpha, il2q;     // il2q = 1 / (4 lambda^2)
    int model;                  // tensor variant (GEN kernels only)
    int up;                     // stream the segment bottom up (eed4_pair.h only)
};

// mu1 = g(x) and mu3 of the tensor variants, x = (s/lambda)^2: the
// diffusivities of Table 7 (Geman-Reynolds scaled to g(0) = 1) and the mu3
// choices of Sec. 3.1 (geometric mean, arithmetic mean or maximum of mu1 and
// mu2 = 1).  model = diffusivity | rule << 4, uniform over the launch.
__device__ __forceinline__ void model_mu(float x, int model, float &mu1, float &mu3)
{
#pragma clang fp contract(off)
    const int diff = model & 0xf, rule = model >> 4;
    const float d = 1.0f + x;
    float g;
    if (diff == kDiffPeronaMalik) {
        g = __builtin_amdgcn_rcpf(d);
    } else if (diff == kDiffPeronaMalikExp) {
        // exp(-x) = 2^(-x log2 e) on the hardware exp2 (1 ulp): two instructions
        // instead of the library's range reduction
        g = __builtin_amdgcn_exp2f(-x * 1.44269504088896341f);
    } else if (diff == kDiffGemanReynolds) {
        const float r = __builtin_amdgcn_rcpf(d);
        g = r * r;
    } else {
        g = __builtin_amdgcn_rsqf(d);
    }
    mu1 = g;
    mu3 = rule == kMu3Arithmetic ? 0.5f * (1.0f + g)
        : rule == kMu3Max        ? 1.0f
                                 : __builtin_amdgcn_sqrtf(g);
}

// model_mu for N points at once: one uniform branch per field for all of them,
// so that the points' arithmetic stays in one block each and can interleave.
template <int N>
__device__ __forceinline__ void model_mu_rows(const float (&x)[N], int model, float (&mu1)[N],
                                              float (&mu3)[N])
{
#pragma clang fp contract(off)
    const int diff = model & 0xf, rule = model >> 4;
    if (diff == kDiffPeronaMalik) {
#pragma unroll
        for (int i = 0; i < N; ++i) mu1[i] = __builtin_amdgcn_rcpf(1.0f + x[i]);
    } else if (diff == kDiffPeronaMalikExp) {
#pragma unroll
        for (int i = 0; i < N; ++i) mu1[i] = __builtin_amdgcn_exp2f(-x[i] * 1.44269504088896341f);
    } else if (diff == kDiffGemanReynolds) {
#pragma unroll
        for (int i = 0; i < N; ++i) {
            const float r = __builtin_amdgcn_rcpf(1.0f + x[i]);
            mu1[i] = r * r;
        }
    } else {
#pragma unroll
        for (int i = 0; i < N; ++i) mu1[i] = __builtin_amdgcn_rsqf(1.0f + x[i]);
    }
    if (rule == kMu3Arithmetic) {
#pragma unroll
        for (int i = 0; i < N; ++i) mu3[i] = 0.5f * (1.0f + mu1[i]);
    } else if (rule == kMu3Max) {
#pragma unroll
        for (int i = 0; i < N; ++i) mu3[i] = 1.0f;
    } else {
#pragma unroll
        for (int i = 0; i < N; ++i) mu3[i] = __builtin_amdgcn_sqrtf(mu1[i]);
    }
}

// Raw buffer resource over the `bytes` bytes from `base` (gfx9 descriptor:
// stride 0, no swizzle).  A load at a byte offset at or beyond `bytes` reads 0
// and a store there is dropped: lanes without an output pixel use kOffNone.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t buffer_rsrc(const void *base, unsigned bytes)
{
    // The empty asm makes the size and flag words opaque, so resources with
    // equal words get SGPRs of their own: otherwise the compiler keeps one copy
    // and rebuilds the four-register descriptor before every access in the loop.
    int flags = 0x00020000;
    asm volatile("" : "+s"(bytes), "+s"(flags));
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(base), (short)0, (int)bytes,
                                             flags);
}
constexpr unsigned kOffNone = 0x80000000u;

__device__ __forceinline__ float buf_f32(__amdgpu_buffer_rsrc_t r, unsigned voff, unsigned soff)
{
    return __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(r, voff, soff, 0));
}

// A wave-uniform row index in a scalar register.  The compiler may form such a
// value with a vector instruction (v_min3), and would then wrap every access
// that takes it as its scalar offset in a loop over distinct lane values.
__device__ __forceinline__ unsigned uniform_row(int r)
{
    return (unsigned)__builtin_amdgcn_readfirstlane(r);
}

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ f32x4 buf_f32x4(__amdgpu_buffer_rsrc_t r, unsigned voff)
{
    return __builtin_bit_cast(f32x4, (u32x4)__builtin_amdgcn_raw_buffer_load_b128(r, voff, 0, 0));
}

// The Gaussian taps in vector registers (R + 1 of them: the kernel is
// symmetric, w[j] = w[2R - j]).  A vector instruction with a scalar-register
// operand issues every 4.15 cycles, one with vector registers only every 2.4
// to 2.6 (measured, 2 to 8 waves a SIMD), and the two passes are a third of
// the step's instructions.
template <int R>
__device__ __forceinline__ void vector_weights(const float *w, float (&wv)[2 * R + 1])
{
#pragma unroll
    for (int j = 0; j <= R; ++j) {
        wv[j] = w[j];
        asm volatile("" : "+v"(wv[j]));
        wv[2 * R - j] = wv[j];
    }
}

// Image row of consecutive stream rows under the half-sample mirror: the row
// moves in direction dir; at an edge it repeats once and the direction flips.
struct RowTrack {
    int y, dir;
    __device__ __forceinline__ void init(int y0, int H)
    {
        y = mirror_reflect(y0, H);
        const int k = y0 >= 0 ? y0 / H : -1 - (-1 - y0) / H;   // mirror copy index
        dir = (k & 1) ? -1 : 1;
    }
    __device__ __forceinline__ void next(int H)
    {
        int nx = y + dir;
        if ((unsigned)nx >= (unsigned)H) {
            dir = -dir;
            nx = y;
        }
        y = nx;
    }
};

// Global loads of one stream row: u^k of the row itself (the lane's column and
// one right-halo column), and u^{k-1}, the mask and the residual reference of
// the output row it serves.
struct StripRow {
    float a, b, pv, rf;
    unsigned mk;
};

// Addressing: every plane is seen through a buffer resource based at image
// row b0 = max(Y0 - h, 0) (the lowest row a needed value comes from) and
// covering nb = min(H - b0, NROW) rows, so a row offset is one 32-bit scalar
// (rows_addressable(NROW)) and the per-lane column offsets stay fixed for the
// whole strip.

template <int R, bool RES, int ROWS, bool GEN = false, bool VST = false>
__device__ __forceinline__ void strip_step(float *ring, const StripArgs &s,
                                           const float (&w)[2 * kRMax + 1], double *partial)
{
    using G = StripGeo<R, ROWS>;
    constexpr int P = G::P, U = G::U, D = G::D, CS = G::CS;
    const int lane = threadIdx.x & 63;
    const int H = s.H, W = s.W;
    const unsigned W4 = 4u * (unsigned)W;
    if constexpr (kLdsSentinel) sentinel_fill_wave(ring, G::LDS);

    const int ystart = s.Y0 - G::h;                           // image row of stream row 0
    const int b0 = ystart > 0 ? ystart : 0;
    const int nb = (H - b0 < G::NROW) ? H - b0 : G::NROW;
    const size_t base = (size_t)b0 * W;
    const __amdgpu_buffer_rsrc_t rs_u = buffer_rsrc(s.ucur + base, (unsigned)nb * W4);
    const __amdgpu_buffer_rsrc_t rs_p = buffer_rsrc(s.uprev + base, (unsigned)nb * W4);
    const __amdgpu_buffer_rsrc_t rs_o = buffer_rsrc(s.uout + base, (unsigned)nb * W4);
    const __amdgpu_buffer_rsrc_t rs_m = buffer_rsrc(s.mask + base, (unsigned)nb * (unsigned)W);
    __amdgpu_buffer_rsrc_t rs_r = rs_p;
    if constexpr (RES) rs_r = buffer_rsrc(s.ref + base, (unsigned)nb * W4);
    __amdgpu_buffer_rsrc_t rs_v = rs_o;
    if constexpr (VST) rs_v = buffer_rsrc(s.vout + base, (unsigned)nb * W4);

    // Staged columns (fixed for the whole strip): staged column j is image
    // column X0-2-R+j.  Lane l stages j = l, and the 2R right-halo columns
    // j = 64 .. 63+2R go to lane l = j - 64 mod 2R (lanes with the same halo
    // column load and write the same value).
    const int lb = R > 0 ? lane % (2 * R > 0 ? 2 * R : 1) : 0;
    const unsigned cb = 4u * (unsigned)mirror_reflect(s.X0 - 2 - R + 64 + lb, W);
    const int cl = s.X0 - 2 + lane;                           // this lane's image column
    const unsigned ca = 4u * (unsigned)mirror_reflect(cl - R, W);
    const bool out_col = lane >= 2 && lane < 62 && cl < W;
    const unsigned vo4 = out_col ? 4u * (unsigned)cl : kOffNone;
    const unsigned vo1 = out_col ? (unsigned)cl : kOffNone;
    float *col = ring + (lane + 1) * CS;                     // ring column of staged column l
    float *bcol = ring + (64 + lb + 1) * CS;                 // right-halo column it stages

    float win[P];                                        // x-pass values, row i in slot i % P
#pragma unroll
    for (int j = 0; j < P; ++j) win[j] = 0.0f;
    float v_m1 = 0.0f, v_m2 = 0.0f;                      // v at rows g, g-1 (before update)
    float txx_p = 0.0f, tyy_p = 0.0f, tyy_pp = 0.0f;     // T at rows g-1 (and g-2 for Tyy)
    float z_p = 0.0f, z_pp = 0.0f;                       // Txy(c+1)-Txy(c-1) at rows g-1, g-2
    float uc_p = 0.0f;                                   // u^k(g-1, c)
    double d2 = 0.0, n2 = 0.0;

    // the next row to prefetch: its mirrored image row and the output row it serves
    RowTrack ty;
    ty.init(ystart, H);
    int on = ystart - (R + 2);

    // Loads run two stream rows ahead, always in the same order, so waiting
    // for one row never waits for a later row's loads.
    auto prefetch = [&](StripRow &r) {
        const unsigned su = (unsigned)((ty.y > b0 ? ty.y : b0) - b0) * W4;
        r.a = buf_f32(rs_u, ca, su);
        if constexpr (R > 0) r.b = buf_f32(rs_u, cb, su);
        int oc = on < b0 ? b0 : on;                      // clamped; unused rows are not stored
        oc = oc > H - 1 ? H - 1 : oc;
        const unsigned ro = (unsigned)(oc - b0);
        r.pv = buf_f32(rs_p, vo4, ro * W4);
        r.mk = __builtin_amdgcn_raw_buffer_load_b8(rs_m, vo1, ro * (unsigned)W, 0);
        if constexpr (RES) r.rf = buf_f32(rs_r, vo4, ro * W4);
        ty.next(H);
        ++on;
    };
    StripRow r0, r1;
    r0.b = r1.b = 0.0f;
    r0.rf = r1.rf = 0.0f;
    prefetch(r0);
    prefetch(r1);

    // The Hessian of u at row g needs u(x-1), u(x), u(x+1) at rows g-1, g, g+1.
    // Segments of >= 64 rows (about 4 waves a SIMD, registers to spare) keep them
    // per staged row, as u(x), u(x-1) + u(x+1) and u(x+1) - u(x-1), in registers
    // indexed like the ring (slot i % D), from the x-pass taps R-1, R, R+1 of row i;
    // the shorter strips, which need 8 waves a SIMD, read them back from the ring.
    constexpr bool HREG = ROWS >= 64;
    constexpr int HD = HREG ? D : 1;
    float hc[HD], hs[HD], hd[HD];
#pragma unroll
    for (int j = 0; j < HD; ++j) hc[j] = hs[j] = hd[j] = 0.0f;

    // stage one row of u^k into ring row rr and take its x pass into window slot ws
    auto stage_xpass = [&](const StripRow &cur, int rr, int ws) {
        col[rr] = cur.a;
        if constexpr (R > 0) bcol[rr] = cur.b;
        wave_lds_sync();
        float acc = w[0] * col[rr];
#pragma unroll
        for (int j = 1; j <= 2 * R; ++j) acc = fmaf(w[j], col[j * CS + rr], acc);
        win[ws] = acc;
        if constexpr (HREG) {
            const float l = col[(R - 1) * CS + rr], c = col[R * CS + rr], r = col[(R + 1) * CS + rr];
            hc[rr] = c;
            hs[rr] = l + r;
            hd[rr] = xdiff(l, r);
        }
    };

    // ---- prologue: stage rows 0 .. 2R-1 and their x pass ----
#pragma unroll
    for (int i = 0; i < 2 * R; ++i) {
        const StripRow cur = r0;
        r0 = r1;
        prefetch(r1);
        stage_xpass(cur, i % D, i % P);
    }

    // iterations up to the image's last row (the tall segments end there; a constant
    // bound with an early exit: with a variable bound the compiler took up to 275
    // registers)
    const int below = H - s.Y0;
    const int M = HREG && below < G::OH ? (below + 4 + U - 1) / U : G::M;
#pragma unroll 1
    for (int it = 0; it < G::M; ++it) {
        // Issue priority falls as the wave moves down its segment, so waves
        // that are behind get the SIMD first and all waves progress together.
        // With the default oldest-first order the early waves finish first and
        // the launch ends with few waves per SIMD to hide latency (about 4.4 of
        // 8 resident on average at 4096^2); this schedule took 64-row strips
        // from 49 to 44.5 us there, with bitwise the same results.
        // The adjoint's recompute steps (VST) stay at the lowest priority: they
        // run beside the reverse steps, which are the critical path.
        if constexpr (!VST) {
            const int left = M - it;
            if (left >= 4) __builtin_amdgcn_s_setprio(3);
            else if (left == 3) __builtin_amdgcn_s_setprio(2);
            else if (left == 2) __builtin_amdgcn_s_setprio(1);
            else __builtin_amdgcn_s_setprio(0);
        }
#pragma unroll
        for (int ph = 0; ph < U; ++ph) {
            const int i = 2 * R + it * U + ph;           // stream row (wave-uniform)
            const StripRow cur = r0;
            r0 = r1;
            prefetch(r1);                                 // mirrored: always valid rows

            // ---- S1: stage u^k row i and take the x pass ----
            stage_xpass(cur, (2 * R + ph) % D, (2 * R + ph) % P);   // constants once unrolled

            // ---- S2: y pass at stream row i - R ----
            // stream row i - R + j is in slot (ph + R + j) % P
            const float v = ypass_sym<R>(w, [&](int j) { return win[(ph + R + j) % P]; });

            // ---- S3: gradient, tensor, Hessian, contraction at row g = i - R - 1 ----
            // (the first rows of the loop produce values that only feed unstored rows)
            const float vo = v_m2;                                            // v at row g - 1
            const float gxs = from_next_lane(v_m1) - from_prev_lane(v_m1);   // 2 gx
            const float gys = v - v_m2;                                       // 2 gy
            // rows g-1, g, g+1 are in ring slots sm, sg, sp; this lane's column
            // is staged column l + R
            const int sm = (R - 2 + ph + D) % D, sg = (R - 1 + ph + D) % D, sp = (R + ph) % D;
            float uc, hxx, hyy, hxy;
            if constexpr (HREG) {
                uc = hc[sg];
                hxx = second_diff_sum(hs[sg], uc);
                hyy = second_diff(hc[sm], uc, hc[sp]);
                hxy = mixed_diff(hd[sp], hd[sm]);
            } else {
                const float *um = col + R * CS + sm;
                const float *u0 = col + R * CS + sg;
                const float *up = col + R * CS + sp;
                uc = u0[0];
                hxx = second_diff(u0[-CS], uc, u0[CS]);
                hyy = second_diff(um[0], uc, up[0]);
                hxy = mixed_diff(xdiff(up[-CS], up[CS]), xdiff(um[-CS], um[CS]));
            }

            const float s2 = grad2_sq(gxs, gys);                              // 4 |grad|^2
            float mu1, mu3;
            if constexpr (GEN) {
                model_mu(s2 * s.il2q, s.model, mu1, mu3);
            } else {                                     // FOEED: Charbonnier, sqrt
                foeed_mu(s2, s.il2q, mu1, mu3);
            }
            float txx, tyy, txy;
            contract(gxs, gys, s2, mu1, mu3, hxx, hyy, hxy, txx, tyy, txy);
            v_m2 = v_m1;
            v_m1 = v;

            // ---- S4: output row o = g - 1 (stream row i - R - 2) ----
            const float z = from_next_lane(txy) - from_prev_lane(txy);
            const int o = ystart + (i - R - 2);
            if (i >= 2 * G::h && o < H) {                // the first output row is Y0
                const unsigned ro = (unsigned)(o - b0) * W4;
                const float sxx = from_prev_lane(txx_p) + from_next_lane(txx_p);
                const float pu = outer_div(txx_p, tyy_p, sxx, tyy_pp + tyy, z, z_pp);
                const float un = fsi_update(pu, uc_p, cur.pv, s.tau, s.alpha, cur.mk != 0);
                if constexpr (RES) {
                    // columns without a pixel read 0 for the reference; add 0
                    const double du = out_col ? (double)un : 0.0;
                    const double dd = du - (double)cur.rf;
                    d2 = fma(dd, dd, d2);
                    n2 = fma(du, du, n2);
                }
                __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(un), rs_o, vo4, ro, 0);
                if constexpr (VST)
                    __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(vo), rs_v, vo4, ro, 0);
            }
            tyy_pp = tyy_p;
            tyy_p = tyy;
            txx_p = txx;
            z_pp = z_p;
            z_p = z;
            uc_p = uc;
        }
        if constexpr (HREG)
            if (it + 1 == M) break;
    }
    if constexpr (RES) {
        for (int off = 32; off > 0; off >>= 1) {
            d2 += __shfl_down(d2, off, 64);
            n2 += __shfl_down(n2, off, 64);
        }
        // lane 0 holds the sums; every lane stores that same value (no
        // lane-dependent branch at the end of a batched queue-loop body)
        const double d2s = lane0_double(d2), n2s = lane0_double(n2);
        partial[0] = d2s;
        partial[1] = n2s;
    }
}

}  // namespace eed4
