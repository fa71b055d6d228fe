// Device code of one fused FOEED/FSI inner step on a tall strip, one wavefront
// per strip, two adjacent columns per lane: the strip pipeline of eed4_strip.h
// (stages S1..S4, bitwise the same arithmetic per pixel) for large images.
//
// A step of 4096^2 at R = 6 is bound by instruction issue, of 8192^2 by memory.
// Against one column per lane: a row of two columns takes one global load, one
// store, one LDS write and R + 1 LDS reads of 8 bytes, and half the DPP shifts;
// the 2R halo columns of four rows are fetched by one instruction of all 64
// lanes; the taps are in vector registers; 124 of 128 columns are outputs, not
// 60 of 64; and the number of rows is a launch argument, so the host can pick a
// segment height that fills the SIMDs evenly (fit_strip_rows).
// Measured (kernels alone), R = 6, one column per lane (64-row segments) against this:
// 4096^2 50.6 -> 47.9 us, 8192^2 213 -> 196 us; R = 3 45.3 -> 42.0, 221 -> 190.
#pragma once

#include "eed4_strip.h"

namespace eed4 {

typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef unsigned u32x2 __attribute__((ext_vector_type(2)));

// The stream is taken in groups of four rows (the halo fetch).  The LDS ring
// holds the last D rows column-pair-major: pair p of ring row r at p * DS + r,
// DS odd, so the lanes' 8-byte accesses spread over the banks and every access
// is a compile-time offset from the lane's own pair.
template <int R>
struct PairGeo {
    static constexpr int P = 2 * R + 1;                              // y window length
    static constexpr int U = ((P > R + 2 ? P : R + 2) + 3) / 4 * 4;  // unroll = window slots
    static constexpr int D = R <= 6 && U % 8 == 0 ? 8 : U;           // ring rows (>= R + 2)
    static constexpr int h = R + 2;                                  // input halo
    static constexpr int PR = (2 * R + 3) / 4 * 4;                   // prologue rows
    static constexpr int LEAD = PR - 2 * R;                          // of which unused ahead
    static constexpr int SW = 124;                                   // output columns per wave
    static constexpr int NP = (R + 1) / 2;                           // halo pairs on each side
    static constexpr int DS = D | 1;                                 // ring stride of a pair
    static constexpr int LDS = 2 * (64 + 2 * NP) * DS;               // floats of LDS per wave
    static_assert(D >= R + 2 && U % D == 0 && D % 4 == 0 && 2 * R <= 16, "ring geometry");
    static_assert(rows_addressable(136 + 4 + PR), "row offsets");    // 136: the most rows
};

// Global loads of one stream row: the lane's two columns of u^k, and u^{k-1},
// the mask and the residual reference of the output row it serves.
struct PairRow {
    f32x2 a, pv, rf;
    unsigned m0, m1;        // mask bytes (one 16-bit load into m0 unless EDGE)
};

// Direction: callers stream odd segments bottom up and even ones top down, so
// the 2h rows two neighbouring segments share are read by both at nearly the
// same time and the second read usually hits in L2 (8192^2, 48-row segments:
// 209.7 us all down, 205.0 alternating; 28-row 221.5 and 216.6; 4096^2 level).
// The stencils are symmetric in y: streaming up only negates the y-odd
// quantities (G_y, u_xy, T_xy and its x differences) exactly, and the y pass is
// symmetric, so u^{k+1} (and the kept v) are bitwise those of the downward
// stream; only the FP64 residual partials add the rows in the other order.
//
// `rows` output rows (a multiple of 4) from s.Y0.  EDGE: the strip touches the
// left or right image border, or its columns pass it: single-column accesses at
// mirrored or dropped columns.  The 8- and 2-byte accesses of the other strips
// need only 4- and 1-byte alignment (any width, any plane address).
template <int R, bool RES, bool VST, bool EDGE>
__device__ __forceinline__ void pair_step(float *ring, const StripArgs &s,
                                          const float (&w)[2 * kRMax + 1], int rows,
                                          double *partial)
{
    using G = PairGeo<R>;
    constexpr int U = G::U, D = G::D, DS = G::DS, NP = G::NP, h = G::h, PR = G::PR;
    const int lane = threadIdx.x & 63;
    const int H = s.H, W = s.W;
    const unsigned W4 = 4u * (unsigned)W;
    if constexpr (kLdsSentinel) sentinel_fill_wave(ring, G::LDS);

    // planes, row offsets and direction as in strip_step
    const int nrow = rows + 4 + PR;                           // stream rows, a multiple of 4
    const int ybase = s.Y0 - h - (s.up ? 0 : G::LEAD);        // lowest streamed row
    const int dir = s.up ? -1 : 1;
    const int ystart = s.up ? ybase + nrow - 1 : ybase;
    const int b0 = ybase > 0 ? ybase : 0;
    const int nb = (H - b0 < nrow) ? H - b0 : nrow;
    const size_t base = (size_t)b0 * W;
    const __amdgpu_buffer_rsrc_t rs_u = buffer_rsrc(s.ucur + base, (unsigned)nb * W4);
    const __amdgpu_buffer_rsrc_t rs_p = buffer_rsrc(s.uprev + base, (unsigned)nb * W4);
    const __amdgpu_buffer_rsrc_t rs_o = buffer_rsrc(s.uout + base, (unsigned)nb * W4);
    const __amdgpu_buffer_rsrc_t rs_m = buffer_rsrc(s.mask + base, (unsigned)nb * (unsigned)W);
    __amdgpu_buffer_rsrc_t rs_r = rs_p;
    if constexpr (RES) rs_r = buffer_rsrc(s.ref + base, (unsigned)nb * W4);
    __amdgpu_buffer_rsrc_t rs_v = rs_o;
    if constexpr (VST) rs_v = buffer_rsrc(s.vout + base, (unsigned)nb * W4);

    // The lane's columns c0, c0 + 1; lanes 1 .. 62 hold outputs.
    const int c0 = s.X0 - 2 + 2 * lane;
    const bool ol = lane >= 1 && lane < 63;
    const bool out0 = ol && (!EDGE || c0 < W), out1 = ol && (!EDGE || c0 + 1 < W);
    unsigned ua, ub = 0, o0, o1 = 0, q0, q1 = 0;
    if constexpr (EDGE) {
        ua = 4u * (unsigned)mirror_reflect(c0, W);
        ub = 4u * (unsigned)mirror_reflect(c0 + 1, W);
        o0 = out0 ? 4u * (unsigned)c0 : kOffNone;
        o1 = out1 ? 4u * (unsigned)(c0 + 1) : kOffNone;
        q0 = out0 ? (unsigned)c0 : kOffNone;
        q1 = out1 ? (unsigned)(c0 + 1) : kOffNone;
    } else {
        ua = 4u * (unsigned)c0;
        o0 = ol ? 4u * (unsigned)c0 : kOffNone;
        q0 = ol ? (unsigned)c0 : kOffNone;
    }
    // Halo: 16 lanes to a row of the group; k < R the left columns, then the
    // right ones; lanes past 2R repeat one (same address, same value).
    const int hrow = lane >> 4;
    const int hk = (lane & 15) < 2 * R ? lane & 15 : 0;
    const int hcol = hk < R ? s.X0 - 2 - R + hk : s.X0 + 126 + hk - R;
    const int hslot = hk < R ? 2 * NP - R + hk : 2 * NP + 128 + hk - R;
    const unsigned hoff = 4u * (unsigned)mirror_reflect(hcol, W);

    float wv[2 * R + 1];
    vector_weights<R>(w, wv);
    float tau = s.tau, alpha = s.alpha, il2q = s.il2q;
    asm volatile("" : "+v"(tau), "+v"(alpha), "+v"(il2q));

    float win[2][U];                                     // x-pass values, row i in slot i % U
#pragma unroll
    for (int j = 0; j < U; ++j) win[0][j] = win[1][j] = 0.0f;
    float v_m1[2] = {}, v_m2[2] = {};                    // v at rows g, g-1 (before update)
    float txx_p[2] = {}, tyy_p[2] = {}, tyy_pp[2] = {};  // T at rows g-1 (and g-2 for Tyy)
    float z_p[2] = {}, z_pp[2] = {};                     // Txy(c+1)-Txy(c-1) at rows g-1, g-2
    float uc_p[2] = {};                                  // u^k(g-1, c)
    // u(x), u(x-1) + u(x+1), u(x+1) - u(x-1) at rows g and g-1
    float hc_m[2] = {}, hc_0[2] = {}, hs_0[2] = {}, hd_m[2] = {}, hd_0[2] = {};
    double d2 = 0.0, n2 = 0.0;

    RowTrack ty;                                         // next row to prefetch
    ty.init(ystart, H);
    if (s.up) ty.dir = -ty.dir;
    unsigned sg[4];                                      // row offsets of the next group
    auto track4 = [&]() {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            sg[j] = uniform_row((ty.y > b0 ? ty.y : b0) - b0) * W4;
            ty.next(H);
        }
    };
    auto halo = [&]() -> float {
        const unsigned o = hrow == 0 ? sg[0] : hrow == 1 ? sg[1] : hrow == 2 ? sg[2] : sg[3];
        return buf_f32(rs_u, hoff + o, 0);
    };
    int on = ystart - dir * h;                           // output row the next prefetch serves
    auto prefetch = [&](PairRow &r, unsigned su) {
        int oc = on < b0 ? b0 : on;                      // clamped; unused rows are not stored
        oc = oc > H - 1 ? H - 1 : oc;
        const unsigned ro = (unsigned)(oc - b0);
        if constexpr (EDGE) {
            r.a = f32x2{buf_f32(rs_u, ua, su), buf_f32(rs_u, ub, su)};
            r.pv = f32x2{buf_f32(rs_p, o0, ro * W4), buf_f32(rs_p, o1, ro * W4)};
            if constexpr (RES)
                r.rf = f32x2{buf_f32(rs_r, o0, ro * W4), buf_f32(rs_r, o1, ro * W4)};
            r.m0 = __builtin_amdgcn_raw_buffer_load_b8(rs_m, q0, ro * (unsigned)W, 0);
            r.m1 = __builtin_amdgcn_raw_buffer_load_b8(rs_m, q1, ro * (unsigned)W, 0);
        } else {
            r.a = __builtin_bit_cast(
                f32x2, (u32x2)__builtin_amdgcn_raw_buffer_load_b64(rs_u, ua, su, 0));
            r.pv = __builtin_bit_cast(
                f32x2, (u32x2)__builtin_amdgcn_raw_buffer_load_b64(rs_p, o0, ro * W4, 0));
            if constexpr (RES)
                r.rf = __builtin_bit_cast(
                    f32x2, (u32x2)__builtin_amdgcn_raw_buffer_load_b64(rs_r, o0, ro * W4, 0));
            r.m0 = __builtin_amdgcn_raw_buffer_load_b16(rs_m, q0, ro * (unsigned)W, 0);
            r.m1 = 0;
        }
        on += dir;
    };
    // rows are fetched two ahead of their use, halos a group ahead
    PairRow r0, r1;
    r0.rf = r1.rf = f32x2{0.0f, 0.0f};
    track4();
    float hv = halo();
    unsigned sc0 = sg[2], sc1 = sg[3];                   // rows 2, 3 of the current group
    prefetch(r0, sg[0]);
    prefetch(r1, sg[1]);
    track4();

    f32x2 *own = (f32x2 *)ring + (NP + lane) * DS;       // own pair of ring row 0
    float *hput = ring + (hslot >> 1) * 2 * DS + (hslot & 1) + 2 * hrow;
    // the halos of four rows into the ring, from ring row rr on.  (The rows they
    // replace may still be read as the outer Hessian neighbours of the strip's
    // first and last column, whose tensors no output uses.)
    auto begin_group = [&](int rr) {
        if constexpr (R > 0) {
            hput[2 * rr] = hv;
            hv = halo();
        }
    };
    auto take = [&](int j) {                             // row j of a group
        const PairRow cur = r0;
        r0 = r1;
        prefetch(r1, j == 0 ? sc0 : j == 1 ? sc1 : sg[j - 2]);
        if (j == 3) {
            sc0 = sg[2];
            sc1 = sg[3];
            track4();
        }
        return cur;
    };
    // stage one row of u^k into ring row rr and take its x pass into window slot ws
    auto stage_xpass = [&](const PairRow &cur, int rr, int ws) {
        f32x2 *row = own + rr;
        row[0] = cur.a;
        wave_lds_sync();
        float x[4 * NP + 2];
#pragma unroll
        for (int j = 0; j < 2 * NP + 1; ++j) {
            const f32x2 t = j == NP ? cur.a : row[(j - NP) * DS];
            x[2 * j] = t.x;
            x[2 * j + 1] = t.y;
        }
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            float acc = wv[0] * x[2 * NP - R + q];
#pragma unroll
            for (int j = 1; j <= 2 * R; ++j) acc = fmaf(wv[j], x[2 * NP - R + q + j], acc);
            win[q][ws] = acc;
        }
    };

#pragma unroll
    for (int i = 0; i < PR; ++i) {
        if (i % 4 == 0) begin_group(i % D);
        const PairRow cur = take(i % 4);
        stage_xpass(cur, i % D, i % U);
    }

    int i = PR, left = rows + 4;
#pragma unroll 1
    for (;;) {
        // issue priority falls as the wave moves down its segment (strip_step)
        if constexpr (!VST) {
            if (left >= 4 * U) __builtin_amdgcn_s_setprio(3);
            else if (left >= 3 * U) __builtin_amdgcn_s_setprio(2);
            else if (left >= 2 * U) __builtin_amdgcn_s_setprio(1);
            else __builtin_amdgcn_s_setprio(0);
        }
#pragma unroll
        for (int ph = 0; ph < U; ++ph) {
            if (ph % 4 == 0) begin_group((PR + ph) % D);
            const PairRow cur = take(ph % 4);

            // ---- S1, S2: x pass of stream row i + ph, y pass of row i + ph - R ----
            stage_xpass(cur, (PR + ph) % D, (PR + ph) % U);
            float v[2];
#pragma unroll
            for (int q = 0; q < 2; ++q)
                v[q] = ypass_sym<R>(wv, [&](int j) { return win[q][(PR + ph - R + j + U) % U]; });

            // ---- S3: gradient, Hessian, tensor, contraction at row g = i + ph - R - 1 ----
            const f32x2 *hr = own + (PR + ph - R + D) % D;        // row g + 1
            const f32x2 c = hr[0];
            float lf, rt;
            if constexpr (R > 0) {
                lf = hr[-DS].y;
                rt = hr[DS].x;
            } else {                                              // no halo pairs in the ring
                lf = from_prev_lane(c.y);
                rt = from_next_lane(c.x);
            }
            const float hc_p[2] = {c.x, c.y};
            const float hs_p[2] = {lf + c.y, c.x + rt};
            const float hd_p[2] = {xdiff(lf, c.y), xdiff(c.x, rt)};
            const f32x2 vo = {v_m2[0], v_m2[1]};                  // v at row g - 1
            float txx[2], tyy[2], txy[2];
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                const float gxs = q == 0 ? v_m1[1] - from_prev_lane(v_m1[1])
                                         : from_next_lane(v_m1[0]) - v_m1[0];   // 2 gx
                const float gys = v[q] - v_m2[q];                               // 2 gy
                const float hxx = second_diff_sum(hs_0[q], hc_0[q]);
                const float hyy = second_diff(hc_m[q], hc_0[q], hc_p[q]);
                const float hxy = mixed_diff(hd_p[q], hd_m[q]);
                const float s2 = grad2_sq(gxs, gys);
                float mu1, mu3;
                foeed_mu(s2, il2q, mu1, mu3);
                contract(gxs, gys, s2, mu1, mu3, hxx, hyy, hxy, txx[q], tyy[q], txy[q]);
            }

            // ---- S4: output row o = g - 1 ----
            const float z[2] = {txy[1] - from_prev_lane(txy[1]), from_next_lane(txy[0]) - txy[0]};
            const int o = ystart + dir * (i + ph - h);
            if (i + ph >= PR + 4 && o < H) {
                const unsigned ro = (unsigned)(o - b0) * W4;
                f32x2 un;
#pragma unroll
                for (int q = 0; q < 2; ++q) {
                    const float sxx = q == 0 ? from_prev_lane(txx_p[1]) + txx_p[1]
                                             : txx_p[0] + from_next_lane(txx_p[0]);
                    const float pu = outer_div(txx_p[q], tyy_p[q], sxx, tyy_pp[q] + tyy[q], z[q],
                                               z_pp[q]);
                    const bool known = EDGE ? (q ? cur.m1 : cur.m0) != 0
                                            : (cur.m0 & (q ? 0xff00u : 0xffu)) != 0;
                    un[q] = fsi_update(pu, uc_p[q], cur.pv[q], tau, alpha, known);
                    if constexpr (RES) {
                        // columns without a pixel read 0 for the reference; add 0
                        const double du = (q ? out1 : out0) ? (double)un[q] : 0.0;
                        const double dd = du - (double)cur.rf[q];
                        d2 = fma(dd, dd, d2);
                        n2 = fma(du, du, n2);
                    }
                }
                if constexpr (EDGE) {
                    __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(un.x), rs_o, o0, ro, 0);
                    __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(un.y), rs_o, o1, ro, 0);
                    if constexpr (VST) {
                        __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(vo.x), rs_v, o0, ro, 0);
                        __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(vo.y), rs_v, o1, ro, 0);
                    }
                } else {
                    __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2, un), rs_o, o0,
                                                          ro, 0);
                    if constexpr (VST)
                        __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2, vo), rs_v,
                                                              o0, ro, 0);
                }
            }
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                v_m2[q] = v_m1[q];
                v_m1[q] = v[q];
                uc_p[q] = hc_0[q];
                hc_m[q] = hc_0[q];
                hc_0[q] = hc_p[q];
                hs_0[q] = hs_p[q];
                hd_m[q] = hd_0[q];
                hd_0[q] = hd_p[q];
                tyy_pp[q] = tyy_p[q];
                tyy_p[q] = tyy[q];
                txx_p[q] = txx[q];
                z_pp[q] = z_p[q];
                z_p[q] = z[q];
            }
            // the segment ends at a group of four rows
            if (ph % 4 == 3) {
                left -= 4;
                if (left <= 0) goto done;
            }
        }
        i += U;
    }
done:
    if constexpr (RES) {
        for (int off = 32; off > 0; off >>= 1) {
            d2 += __shfl_down(d2, off, 64);
            n2 += __shfl_down(n2, off, 64);
        }
        const double d2s = lane0_double(d2), n2s = lane0_double(n2);
        partial[0] = d2s;
        partial[1] = n2s;
    }
}

// The strip at s.X0, s.Y0 of a segment of up to `rows` rows (a multiple of 4).
template <int R, bool RES, bool VST>
__device__ __forceinline__ void pair_strip(float *ring, const StripArgs &s,
                                           const float (&w)[2 * kRMax + 1], int rows,
                                           double *partial)
{
    const int below = (s.H - s.Y0 + 3) / 4 * 4;          // the last segment may be shorter
    const int n = rows < below ? rows : below;
    if (s.X0 < 2 || s.X0 + 126 > s.W)
        pair_step<R, RES, VST, true>(ring, s, w, n, partial);
    else
        pair_step<R, RES, VST, false>(ring, s, w, n, partial);
}

}  // namespace eed4
