// Device code of one fused FOEED/FSI inner step on one output tile.
//
// One workgroup of NTH threads computes a tile of u^{k+1} from u^k (read with
// a halo of R+2 pixels, R = Gaussian radius) and u^{k-1}.  TW lanes hold TW
// consecutive columns, of which the middle TW - 4 are outputs (the contracted
// Hessian T needs one column more on each side and the gradient another); a
// group of TW lanes owns OH consecutive rows, and the NTH / TW groups stack to
// TH rows:
//   A  u^k of the tile and its halo into LDS, 16 bytes a lane (border tiles
//      gather through the half-sample mirror, which realises the Neumann
//      condition, Sec. 2.1); u^{k-1}, mask and cycle start of the group's own
//      outputs into registers, so that their latency hides behind the stages
//   B  x pass of the separable Gaussian presmoothing (Sec. 2.2), four outputs
//      per item from 16-byte LDS reads, each row once per workgroup
//   C  in registers, every row of the group at once: y pass, central-difference
//      gradient of u_sigma, fourth-order diffusion tensor from it (Sec. 3.1),
//      Hessian of u (Sec. 3.3 stencils, mixed term with corrected signs),
//      T = D : H, outer second differences of T (eq. genModel), explicit step,
//      FSI extrapolation (Sec. 3.3) and Dirichlet hold; optionally the FP64
//      cycle residual and the presmoothed image K_sigma * u^k.
// Every intermediate is evaluated on the mirror-extended image, so the halo
// values of T carry the parity the boundary needs and P stays symmetric.
//
// What bounds it: a tile is a chain of a global load, two barriers and about
// OH + 4 rows of dependent arithmetic, and below about a million pixels that
// chain and the launch are the whole time.  Stage C keeps OH + 4 independent
// rows in flight, which the streaming strips cannot, and reads the x pass from
// LDS instead of taking it again for the 2R + 4 halo rows of every group.  Of its
// cycles a wave waits for a load, LDS or a barrier 0.46 on 512^2 (R = 5, 32 x 16),
// 0.32 on 1037x771 (R = 8, 32 x 32) and 0.40 on 1024^2 (64 x 32), and is ready while
// another wave issues 0.17, 0.31 and 0.18; on 4096^2 (R = 6) 0.19 and 0.45.
#pragma once

#include "eed4_internal.h"
#include "eed4_pointwise.h"
#include "eed4_strip.h"

namespace eed4 {

__device__ __forceinline__ int mirror_index(int i, int n)
{
    int p = 2 * n;
    int m = i % p;
    if (m < 0) m += p;
    return m < n ? m : p - 1 - m;
}

// Half-sample mirror of -n <= i < 2n (one reflection at each end: -1 - i == ~i).
// Indices beyond that give a value the caller clamps (nothing needed comes from
// them).
__device__ __forceinline__ int mirror_once(int i, int n)
{
    const int m = i > ~i ? i : ~i;
    const int r = 2 * n - 1 - m;
    return m < r ? m : r;
}

template <int R, int TW, int TH, int NTH = kThreads>
struct TileGeo {
    static constexpr int OH = TH * TW / NTH;              // output rows per lane group
    static_assert(64 % TW == 0 && TW >= 16 && OH >= 1 && OH * (NTH / TW) == TH, "tile shape");
    static constexpr int h = R + 2;                       // input halo
    static constexpr int SW = TW - 4;                     // output columns
    static constexpr int SC = (h + 3) & ~3;               // staged columns left of the outputs
    static constexpr int OFF = SC - h;                    // first tap of lane 0's column
    static constexpr int UH = TH + 2 * h;                 // staged rows
    static constexpr int UWn = SC + TW + (R > 2 ? R - 2 : 0);  // staged columns needed
    static constexpr int UQ = (UWn + 3) / 4;              // 16-byte loads per staged row
    static constexpr int NF4 = (OFF + 4 + 2 * R + 3) / 4; // 16-byte LDS reads per x-pass item
    static constexpr int NQ = TW / 4;                     // x-pass items per row
    static constexpr int UW = 4 * (UQ > NF4 + NQ - 1 ? UQ : NF4 + NQ - 1);   // row stride of u
    static constexpr int NA = UH * UQ, NB = UH * NQ;      // items of stages A and B
    static constexpr int NU = UH * UW, NX = UH * TW;
    static constexpr int SMEM = NU + NX;                  // floats of LDS
    static constexpr int NV = OH + 4, NT = OH + 2;        // rows of v and of T per group
    static constexpr int IA = (NA + NTH - 1) / NTH;       // stage A items per thread
    static_assert(rows_addressable(UH), "row offsets");
};

// Stage A: 16 bytes of u per item, from row y0 / column xs of the mirrored
// image (b0: image row of the resource's base), ...
template <typename G, int NTH>
__device__ __forceinline__ void tile_load(f32x4 (&st)[G::IA], __amdgpu_buffer_rsrc_t rs, int xs,
                                          int y0, int b0, int H, int W)
{
    const unsigned W4 = 4u * (unsigned)W;
    if (H >= G::UH && xs >= 0 && xs + 4 * G::UQ <= W) {
#pragma unroll
        for (int k = 0; k < G::IA; ++k) {
            const int it = threadIdx.x + k * NTH, r = it / G::UQ, q = it - r * G::UQ;
            int y = mirror_once(y0 + r, H);
            y = y < b0 ? b0 : y;
            const unsigned vo = it < G::NA ? (unsigned)(y - b0) * W4 + 4u * (unsigned)(xs + 4 * q)
                                           : kOffNone;
            st[k] = buf_f32x4(rs, vo);
        }
    } else {
        const bool tiny = H < G::UH || W < 4 * G::UQ;     // may need repeated reflection
#pragma unroll
        for (int k = 0; k < G::IA; ++k) {
            const int it = threadIdx.x + k * NTH, r = it / G::UQ, q = it - r * G::UQ;
            int y = tiny ? mirror_index(y0 + r, H) : mirror_once(y0 + r, H);
            y = y < b0 ? b0 : y;
            const unsigned ro = (unsigned)(y - b0) * W4;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int x = xs + 4 * q + e;
                int xm = tiny ? mirror_index(x, W) : mirror_once(x, W);
                xm = xm < 0 ? 0 : xm;
                st[k][e] = buf_f32(rs, it < G::NA ? ro + 4u * (unsigned)xm : kOffNone, 0);
            }
        }
    }
}

// ... and into LDS.
template <typename G, int NTH>
__device__ __forceinline__ void tile_put(float *sU, const f32x4 (&st)[G::IA])
{
#pragma unroll
    for (int k = 0; k < G::IA; ++k) {
        const int it = threadIdx.x + k * NTH, r = it / G::UQ, q = it - r * G::UQ;
        if (it < G::NA) *reinterpret_cast<f32x4 *>(sU + r * G::UW + 4 * q) = st[k];
    }
}

// Stage B: x pass of every staged row, four columns per item.
template <int R, int TW, typename G, int NTH>
__device__ __forceinline__ void tile_xpass(const float *sU, float *sX, const float (&wv)[2 * R + 1])
{
#pragma unroll
    for (int k = 0; k < (G::NB + NTH - 1) / NTH; ++k) {
        const int it = threadIdx.x + k * NTH;
        if (G::NB % NTH == 0 || it < G::NB) {
            const int r = it / G::NQ, q = it % G::NQ;
            const f32x4 *src = reinterpret_cast<const f32x4 *>(sU + r * G::UW + 4 * q);
            float win[4 * G::NF4];
#pragma unroll
            for (int f = 0; f < G::NF4; ++f) {
                const f32x4 t = src[f];
#pragma unroll
                for (int e = 0; e < 4; ++e) win[4 * f + e] = t[e];
            }
            f32x4 o;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                float acc = wv[0] * win[G::OFF + e];
#pragma unroll
                for (int j = 1; j <= 2 * R; ++j) acc = fmaf(wv[j], win[G::OFF + e + j], acc);
                o[e] = acc;
            }
            *reinterpret_cast<f32x4 *>(sX + TW * r + 4 * q) = o;
        }
    }
}

// Accumulates sum (un - ref)^2 and sum un^2 of the tile in FP64 and writes
// them to out[0..1] (thread 0).  Fixed reduction order: deterministic.
template <int NTH = kThreads>
__device__ __forceinline__ void block_sum2(double d2, double n2, double *scratch, double *out)
{
    for (int o = 32; o > 0; o >>= 1) {
        d2 += __shfl_down(d2, o, 64);
        n2 += __shfl_down(n2, o, 64);
    }
    int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    __syncthreads();
    if (lane == 0) {
        scratch[2 * wv] = d2;
        scratch[2 * wv + 1] = n2;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        double a = 0.0, b = 0.0;
        for (int i = 0; i < NTH / 64; ++i) {
            a += scratch[2 * i];
            b += scratch[2 * i + 1];
        }
        out[0] = a;
        out[1] = b;
    }
}

// One tile.  ucur/uprev/uout/ref/mask point at the image (H x W).  ref, when
// not null, is the cycle-start state for the residual (it may equal uout: each
// pixel is read before it is written by the same thread).  GEN: tensor variant
// `model` chosen at run time; VST: also K_sigma * u^k into vout.
template <int R, int TW, int TH, int NTH = kThreads, bool GEN = false, bool VST = false>
__device__ __forceinline__ void step_tile(float *smem, const float *ucur, const float *uprev,
                                          float *uout, const float *ref,
                                          const uint8_t *__restrict__ mask, int H, int W, int ty,
                                          int tx, const float (&w)[2 * kRMax + 1], float tau,
                                          float alpha, float il2q, double *partial, int model = 0,
                                          float *vout = nullptr)
{
    using G = TileGeo<R, TW, TH, NTH>;
    constexpr int OH = G::OH, NV = G::NV, NT = G::NT;
    float *sU = smem, *sX = smem + G::NU;
    const int tid = threadIdx.x, lane = tid % TW;
    int grp = tid / TW;
    if constexpr (TW == 64) grp = __builtin_amdgcn_readfirstlane(grp);
    const int X0 = tx * G::SW, Y0 = ty * TH, Yg = Y0 + grp * OH;
    if constexpr (kLdsSentinel) sentinel_fill_block(smem, G::SMEM);

    // Every plane through a buffer resource based at the lowest row a needed
    // value comes from (rows_addressable(UH)); lanes without
    // an output pixel use an offset beyond it, so they read 0 and store nothing.
    const unsigned W4 = 4u * (unsigned)W;
    const int y0 = Y0 - G::h, b0 = y0 > 0 ? y0 : 0;
    const int nb = H - b0 < G::UH ? H - b0 : G::UH;
    const size_t base = (size_t)b0 * W;
    const __amdgpu_buffer_rsrc_t rs_u = buffer_rsrc(ucur + base, (unsigned)nb * W4);
    const __amdgpu_buffer_rsrc_t rs_p = buffer_rsrc(uprev + base, (unsigned)nb * W4);
    const __amdgpu_buffer_rsrc_t rs_o = buffer_rsrc(uout + base, (unsigned)nb * W4);
    const __amdgpu_buffer_rsrc_t rs_m = buffer_rsrc(mask + base, (unsigned)nb * (unsigned)W);

    // ---- A: loads ----
    f32x4 st[G::IA];
    tile_load<G, NTH>(st, rs_u, X0 - G::SC, y0, b0, H, W);
    const int c = X0 - 2 + lane;                          // this lane's column
    const bool out_col = lane >= 2 && lane < TW - 2 && c < W;
    const unsigned vo4 = out_col ? 4u * (unsigned)c : kOffNone;
    const unsigned vo1 = out_col ? (unsigned)c : kOffNone;
    // byte offsets of the group's rows: scalar where a group is a whole wave
    auto in_row = [&](int j) {
        const int r = (Yg + j < H ? Yg + j : H - 1) - b0;
        return TW == 64 ? uniform_row(r) : (unsigned)r;
    };
    auto load_row = [&](__amdgpu_buffer_rsrc_t rs, int j) {
        return TW == 64 ? buf_f32(rs, vo4, in_row(j) * W4) : buf_f32(rs, vo4 + in_row(j) * W4, 0);
    };
    auto store_row = [&](__amdgpu_buffer_rsrc_t rs, int j, float x) {
        const unsigned ro = (unsigned)(Yg + j - b0) * W4;
        if constexpr (TW == 64) {
            if (Yg + j < H)
                __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(x), rs, vo4, ro, 0);
        } else {
            __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(x), rs,
                                                  Yg + j < H ? vo4 + ro : kOffNone, 0, 0);
        }
    };
    float ep[OH], ef[OH];
    unsigned em[OH];
#pragma unroll
    for (int j = 0; j < OH; ++j) {
        const unsigned ro = in_row(j) * (unsigned)W;
        ep[j] = load_row(rs_p, j);
        em[j] = TW == 64 ? __builtin_amdgcn_raw_buffer_load_b8(rs_m, vo1, ro, 0)
                         : __builtin_amdgcn_raw_buffer_load_b8(rs_m, vo1 + ro, 0, 0);
        ef[j] = 0.0f;
    }
    if (ref) {
        const __amdgpu_buffer_rsrc_t rs_r = buffer_rsrc(ref + base, (unsigned)nb * W4);
#pragma unroll
        for (int j = 0; j < OH; ++j) ef[j] = load_row(rs_r, j);
    }
    tile_put<G, NTH>(sU, st);
    float wv[2 * R + 1], vtau = tau, valpha = alpha, vil2q = il2q;
    vector_weights<R>(w, wv);
    asm volatile("" : "+v"(vtau), "+v"(valpha), "+v"(vil2q));
    __syncthreads();

    tile_xpass<R, TW, G, NTH>(sU, sX, wv);                // ---- B ----
    __syncthreads();

    // ---- C: the group's rows; row j of xw, u and v is image row Yg - h + j,
    // Yg - 2 + j and Yg - 2 + j, row t of T is Yg - 1 + t ----
    double d2 = 0.0, n2 = 0.0;
    if (TW < 64 || Yg < H) {                              // (wave-uniform where TW == 64)
        const float *px = sX + TW * (grp * OH) + lane;
        const float *pu = sU + G::UW * (grp * OH + R) + (G::SC - 2) + lane;
        float xw[NV + 2 * R];
#pragma unroll
        for (int j = 0; j < NV + 2 * R; ++j) xw[j] = px[TW * j];
        float uc[NV], us[NV], ud[NV], v[NV];
#pragma unroll
        for (int j = 0; j < NV; ++j) {
            const float l = pu[G::UW * j - 1], r = pu[G::UW * j + 1];
            uc[j] = pu[G::UW * j];
            us[j] = l + r;
            ud[j] = xdiff(l, r);
            v[j] = ypass_sym<R>(wv, [&](int t) { return xw[j + R + t]; });
        }
        float gxs[NT], gys[NT], s2[NT], mu1[NT], mu3[NT];
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            gxs[t] = from_next_lane(v[t + 1]) - from_prev_lane(v[t + 1]);            // 2 gx
            gys[t] = v[t + 2] - v[t];                                                // 2 gy
            s2[t] = grad2_sq(gxs[t], gys[t]);                                        // 4 |grad|^2
            if constexpr (!GEN) foeed_mu(s2[t], vil2q, mu1[t], mu3[t]);
        }
        if constexpr (GEN) {
            float x[NT];
#pragma unroll
            for (int t = 0; t < NT; ++t) x[t] = s2[t] * vil2q;
            model_mu_rows(x, model, mu1, mu3);
        }
        float txx[NT], tyy[NT], z[NT];
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            const float hxx = second_diff_sum(us[t + 1], uc[t + 1]);
            const float hyy = second_diff(uc[t], uc[t + 1], uc[t + 2]);
            const float hxy = mixed_diff(ud[t + 2], ud[t]);
            float txy;
            contract(gxs[t], gys[t], s2[t], mu1[t], mu3[t], hxx, hyy, hxy, txx[t], tyy[t], txy);
            z[t] = from_next_lane(txy) - from_prev_lane(txy);
        }
        __amdgpu_buffer_rsrc_t rs_v = rs_o;
        if constexpr (VST) rs_v = buffer_rsrc(vout + base, (unsigned)nb * W4);
#pragma unroll
        for (int j = 0; j < OH; ++j) {
            const float sxx = from_prev_lane(txx[j + 1]) + from_next_lane(txx[j + 1]);
            const float pr = outer_div(txx[j + 1], tyy[j + 1], sxx, tyy[j] + tyy[j + 2], z[j + 2],
                                       z[j]);
            const float un = fsi_update(pr, uc[j + 2], ep[j], vtau, valpha, em[j] != 0);
            const bool row = Yg + j < H;
            if (ref) {
                // pixels outside the image read 0 for the reference; add 0
                const double du = row && out_col ? (double)un : 0.0;
                const double dd = du - (row ? (double)ef[j] : 0.0);
                d2 = fma(dd, dd, d2);
                n2 = fma(du, du, n2);
            }
            store_row(rs_o, j, un);
            if constexpr (VST) store_row(rs_v, j, v[j + 2]);
        }
    }
    if (ref) block_sum2<NTH>(d2, n2, reinterpret_cast<double *>(smem), partial);
}

// Workgroup -> tile map that gives each XCD (workgroups are dealt round-robin
// over 8 XCDs) a contiguous run of tiles, so neighbouring tiles, which share
// halo rows, usually meet in the same L2.
__device__ __forceinline__ int xcd_tile(int bid, int nb)
{
    const int nx = 8;
    int q = nb / nx, rem = nb % nx;
    int xcd = bid % nx, idx = bid / nx;
    int base = xcd < rem ? xcd * (q + 1) : rem * (q + 1) + (xcd - rem) * q;
    return base + idx;
}

}  // namespace eed4
