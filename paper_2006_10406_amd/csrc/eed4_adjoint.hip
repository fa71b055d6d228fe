// Adjoint of the FSI evolution (reverse mode), for the gradient of a loss on
// the inpainted image with respect to the known values f and the contrast
// lambda.  The paper states only the forward scheme (Sec. 3.3); the reverse
// recursion below is derived from it.
//
// Forward step k (F(u) = P(u) u, P from the tensor of Sec. 3.1):
//   u^{k+1} = mbar * [alpha_k (u^k - tau F(u^k)) + (1 - alpha_k) u^{k-1}] + m * f
// Reverse step k, given ubar^{k+1}:
//   fbar += m * ubar^{k+1};  r = mbar * ubar^{k+1}
//   ubar^k     += alpha_k (r - tau J_F(u^k)^T r)
//   ubar^{k-1} += (1 - alpha_k) r                (added to ubar^0 when k = 0)
//   lambdabar  += -alpha_k tau <dF/dlambda, r>
// with J_F(u)^T r = P(u) r + C^T q, C = (grad of the presmoothed image) and
// q_p = de_p/dG_p for e_p = (B r)_p : D(G_p) : (B u)_p (B = Hessian).
// Everything is evaluated on the mirror-extended image, which makes every
// transpose exact: q_x comes out odd across vertical borders and even across
// horizontal ones, q_y the reverse.
//
// Two implementations of a reverse step, each one launch that reads the
// presmoothed image K_sigma * u^k, which the forward recompute keeps, instead
// of blurring u^k again:
//  - workgroup tiles: q and P(u) r of the tile and its halo in registers, d =
//    -div q and its x pass through LDS (small and medium problems);
//  - wave strips: a wave streams down a strip and carries every intermediate
//    in registers and per-wave LDS, as the forward strip kernel does (fewer
//    instructions a pixel: large problems).
// Per step, tiles against the best strip: 512^2 (R = 5) 7.7 against 12.3 us,
// 16 x 256^2 (R = 3) 12.8 against 15.6, 1024^2 (R = 6) 14.9 against 22.5,
// 2048^2 (R = 8) 46 against 58, (R = 6) 39 against 38, 4096^2 (R = 6) 146
// against 114.
// Known pixels: r is 0 there, so ubar on a known pixel feeds nothing but fbar.
// Both implementations therefore keep on known pixels the running sum of ubar
// over the reverse steps done so far; fbar is that sum at the end.  lambdabar
// is accumulated per work item across all reverse steps and reduced once.
#include "eed4.h"
#include "eed4_host.h"
#include "eed4_internal.h"
#include "eed4_strip.h"
#include "eed4_tile.h"

#include <cmath>
#include <vector>

namespace eed4 {

// Eigenvalue data of a tensor variant (diffusivities of Table 7, mu3 choices
// of Sec. 3.1) at x = (s/lambda)^2: mu1 = g(x), mu3, their derivatives G1, G3
// with respect to x, and Q1 = (mu1 - 1)/x, Q3 = (mu3 - 1)/x, written so that
// they stay finite at x = 0 (every variant has g(0) = 1).
struct MuData {
    float mu1, mu3, G1, G3, Q1, Q3;
};

__device__ __forceinline__ MuData model_mu_data(float x, int model)
{
    const int diff = model & 0xf, rule = model >> 4;
    const float d = 1.0f + x;
    MuData m;
    if (diff == kDiffPeronaMalik) {                  // (1 + x)^-1
        m.mu1 = __builtin_amdgcn_rcpf(d);
        m.G1 = -m.mu1 * m.mu1;
        m.Q1 = -m.mu1;
    } else if (diff == kDiffPeronaMalikExp) {        // exp(-x)
        m.mu1 = expf(-x);
        m.G1 = -m.mu1;
        m.Q1 = x > 0.0f ? expm1f(-x) / x : -1.0f;
    } else if (diff == kDiffGemanReynolds) {         // (1 + x)^-2
        const float r = __builtin_amdgcn_rcpf(d);
        m.mu1 = r * r;
        m.G1 = -2.0f * m.mu1 * r;
        m.Q1 = -(2.0f + x) * m.mu1;
    } else {                                         // Charbonnier (1 + x)^-1/2
        m.mu1 = __builtin_amdgcn_rsqf(d);
        m.G1 = -0.5f * m.mu1 * m.mu1 * m.mu1;
        m.Q1 = -m.mu1 * m.mu1 * __builtin_amdgcn_rcpf(1.0f + m.mu1);
    }
    if (rule == kMu3Arithmetic) {                    // (mu1 + mu2)/2
        m.mu3 = 0.5f * (1.0f + m.mu1);
        m.G3 = 0.5f * m.G1;
        m.Q3 = 0.5f * m.Q1;
    } else if (rule == kMu3Max) {                    // max(mu1, mu2) = 1
        m.mu3 = 1.0f;
        m.G3 = 0.0f;
        m.Q3 = 0.0f;
    } else {                                         // sqrt(mu1 mu2)
        m.mu3 = __builtin_amdgcn_sqrtf(m.mu1);
        m.G3 = m.mu1 > 0.0f ? 0.5f * m.G1 * __builtin_amdgcn_rcpf(m.mu3) : 0.0f;
        m.Q3 = m.Q1 * __builtin_amdgcn_rcpf(1.0f + m.mu3);
    }
    return m;
}

// Per-point pieces of the adjoint.  (gx, gy) = G = grad u_sigma; A = Hessian
// of r, H = Hessian of u.  Outputs: D(G) : A, q = de/dG and s de/ds with
// e = A : D(G) : H, s = |G|; mu depends on s/lambda only, so de/dlambda =
// -(s/lambda) de/ds, and the 1/lambda goes into the per-step scale.  In the
// gradient frame n = G/|G|, t = n rotated by +90 degrees, e = A:H +
// (mu1 - 1) a1 h1 + 2 (mu3 - 1) a3 h3 with a1 = n.A.n, a3 = t.A.n; d/ds and
// d/dtheta of it give q = (de/ds) n + (1/s)(de/dtheta) t.
template <bool GEN = false>
__device__ __forceinline__ void adjoint_point(float gx, float gy, float inv_lam2, float axx,
                                              float ayy, float axy, float hxx, float hyy,
                                              float hxy, float &txx, float &tyy, float &txy,
                                              float &qx, float &qy, float &sds, int model = 0)
{
#pragma clang fp contract(off)
    const float s2 = fmaf(gx, gx, gy * gy);
    float mu1, mu3;
    MuData md{};
    if constexpr (GEN) {
        md = model_mu_data(s2 * inv_lam2, model);
        mu1 = md.mu1;
        mu3 = md.mu3;
    } else {
        mu1 = __builtin_amdgcn_rsqf(fmaf(s2, inv_lam2, 1.0f));
        mu3 = __builtin_amdgcn_sqrtf(mu1);
    }
    const float rn = __builtin_amdgcn_rsqf(fmaxf(s2, 1e-30f));
    const float s = s2 * rn;                   // |G| (0 when G = 0)
    const float nx = gx * rn, ny = gy * rn;
    const float a = nx * nx, b = ny * ny, c = nx * ny;
    const float amb = a - b, c2 = c + c;
    const float a1 = fmaf(a, axx, fmaf(b, ayy, c2 * axy));
    const float a3 = fmaf(c, ayy - axx, amb * axy);
    const float h1 = fmaf(a, hxx, fmaf(b, hyy, c2 * hxy));
    const float h3 = fmaf(c, hyy - hxx, amb * hxy);
    // D : A
    const float k1 = fmaf(mu1, a1, -a1);         // (mu1 - 1) a1
    const float k3 = fmaf(mu3, a3, -a3);         // (mu3 - 1) a3
    txx = fmaf(k1, a, fmaf(-k3, c2, axx));
    tyy = fmaf(k1, b, fmaf(k3, c2, ayy));
    txy = fmaf(k1, c, fmaf(k3, amb, axy));
    float de_ds, dth;
    if constexpr (GEN) {
        // with x = s^2/lambda^2: d mu/ds = 2 s/lambda^2 dmu/dx and
        // (mu - 1)/s = s/lambda^2 (mu - 1)/x
        const float Y = fmaf(md.G1, a1 * h1, 2.0f * md.G3 * (a3 * h3));
        de_ds = 2.0f * s * inv_lam2 * Y;
        const float at = fmaf(b, axx, fmaf(a, ayy, -c2 * axy));
        const float ht = fmaf(b, hxx, fmaf(a, hyy, -c2 * hxy));
        const float p1 = fmaf(a3, h1, a1 * h3);
        const float p2 = fmaf(at - a1, h3, a3 * (ht - h1));
        dth = 2.0f * s * inv_lam2 * fmaf(md.Q1, p1, md.Q3 * p2);
    } else {
        // derivatives: dmu1/ds = -s mu1^3 / lam^2, dmu3/ds = -s mu1^(5/2) / (2 lam^2)
        const float Fm = (s * inv_lam2) * (mu1 * mu1);            // s mu1^2 / lam^2
        de_ds = -Fm * fmaf(mu1, a1 * h1, mu3 * (a3 * h3));
        // (mu1 - 1)/s = -s mu1^2 / (lam^2 (1 + mu1)), (mu3 - 1)/s = that / (1 + mu3).
        // With a + b = 1 for the unit n, t.A.t - n.A.n = (axx + ayy) - 2 a1 and the same
        // for H; where G = 0 (n = 0) the factor Fm = 0 zeroes the whole term.
        const float rp = __builtin_amdgcn_rcpf(fmaf(-0.5f, mu1, -0.5f) * (1.0f + mu3));  // -2/(..)
        const float p1 = fmaf(a3, h1, a1 * h3);
        const float p2 = fmaf(fmaf(-2.0f, a1, axx + ayy), h3, a3 * fmaf(-2.0f, h1, hxx + hyy));
        dth = (Fm * rp) * fmaf(p1, 1.0f + mu3, p2);
    }
    qx = fmaf(nx, de_ds, -ny * dth);
    qy = fmaf(ny, de_ds, nx * dth);
    sds = s * de_ds;
}

// The rest of a reverse step's arithmetic, shared by its kernels like the point
// quantities above, with contraction off and every fused multiply-add written
// out: all kernel shapes give bitwise the same gradients of f and u_init.
//
// Second differences, of u and r and of D:A, are differences of first differences,
// (f(x+1) - f(x)) - (f(x) - f(x-1)): between neighbours of a smooth field those are
// exact, while f(x-1) + f(x+1) is rounded at the size of f itself.  Lanes and
// rows share the first differences, so the form costs no more instructions.
// Relative L2 error of dL/du_init against FP64, geometric mean of 15 runs of 128^2 to
// 256^2: 4.01e-7 with the sums, 3.98e-7 so (the output's own rounding is most of it).
//
// First difference along x of a value held by consecutive lanes, and the second
// difference from it.  Strips, which have one row in hand, carry the first to the
// next row: a lane shift right after it would wait for the result (28-row strips, five
// radii: 1.018x the time of the sums so, 1.012x carried; tiles, whose rows interleave,
// 0.99x without).
__device__ __forceinline__ float lane_diff(float v)
{
#pragma clang fp contract(off)
    return from_next_lane(v) - v;
}
__device__ __forceinline__ float lane_diff2(float f)
{
#pragma clang fp contract(off)
    return f - from_prev_lane(f);
}
// P(u) r at a pixel from the second differences xx of T_xx and yy of T_yy (T = D:A)
// and zd / zu = T_xy(x+1) - T_xy(x-1) in the rows below and above, ...
__device__ __forceinline__ float adj_outer(float xx, float yy, float zd, float zu)
{
#pragma clang fp contract(off)
    return fmaf(0.5f, zd - zu, xx + yy);
}
// ... d = -div q from q_x(x+1) - q_x(x-1) and q_y(y+1) - q_y(y-1), ...
__device__ __forceinline__ float adj_div(float ex, float ey)
{
#pragma clang fp contract(off)
    return -0.5f * (ex + ey);
}
// ... and the update from pr = P(u) r, cq = C^T q, ubar^{k+1} and ubar^k.  back
// is (1 - alpha) r, which goes to ubar^k itself at k = 0 (keep_back 1, else 0).
__device__ __forceinline__ float adj_update(float pr, float cq, float an, float ac, bool known,
                                            float tau, float alpha, float keep_back, float &back)
{
#pragma clang fp contract(off)
    const float rv = known ? 0.0f : an;
    back = (1.0f - alpha) * rv;
    const float acv = fmaf(keep_back, back, fmaf(alpha, fmaf(-tau, pr + cq, rv), ac));
    return known ? acv + an : acv;                            // known pixel: running sum
}

// ---- fused reverse step on workgroup tiles ----
//
// A group of 64 lanes holds 64 consecutive columns c = X0-2-R .. X0+61-R; the
// NTH / 64 groups stack to QH rows of adjoint point quantities, Y0-1-R ..
// Y0+TH+R, for the 60-2R x TH outputs of the tile:
//   Q  every group forms D:A, q and s de/ds of its OQ rows in registers, from v
//      = K_sigma * u^k, u^k and r = mbar ubar^{k+1} of those rows and the two
//      around them (all loads of the group in flight at once, lane neighbours
//      by DPP); the first and last row's T_yy, x difference of T_xy and q_y go
//      through LDS to the groups above and below
//   D  d = -div q and P(u) r, into LDS
//   X  x pass of d, four columns per item from 16-byte LDS reads
//   F  y pass of d (C^T q) and the reverse update, OF rows per group
// Like the forward tile it is a chain of a load, a few barriers and the
// arithmetic of OQ independent rows; the strips below issue fewer instructions
// a pixel on large images but need one dependent row after the other.  The
// values are formed by the same operations in the same order as there.
template <int R, int NTH, int OQ>
struct AdjTileGeo {
    static constexpr int NG = NTH / 64;
    static constexpr int QH = NG * OQ;                        // rows of q
    static constexpr int TH = QH - 2 * (R + 1);               // output rows
    static constexpr int OF = (TH + NG - 1) / NG;             // output rows per group
    static constexpr int h = R + 2, hc = R + 2;               // input halo, first output lane
    static constexpr int SW = 64 - 2 * hc;
    static constexpr int DH = TH + 2 * R;                     // rows of d
    static constexpr int C4 = (R + 3) / 4, OFF = 4 * C4 - R;  // x-pass window: quads to the left, first tap
    static constexpr int NF4 = (OFF + 4 + 2 * R + 3) / 4;
    static constexpr int Q0 = hc / 4, NQ = (63 - hc) / 4 - Q0 + 1;   // quads with output lanes
    static constexpr int PL = 4 * (C4 > Q0 ? C4 - Q0 : 0);    // pad left of lane 0 in a d row
    static constexpr int DSn = PL + 4 * (Q0 + NQ - 1 - C4 + NF4);
    static constexpr int DS = DSn > PL + 64 ? DSn : PL + 64;  // row stride of d (a multiple of 4)
    static constexpr int NE = 6 * NG * 64, ND = DH * DS, NX = DH * 64, NP = TH * 64;
    static constexpr int LDS = NE + ND + NX + NP;
    static_assert(TH > 0 && rows_addressable(QH + 2), "tile height");
};

// Wave-tree sum of v, then the groups' sums in order; thread 0 writes scale * sum.
template <int NG>
__device__ __forceinline__ void group_sum(float v, float *scratch, float scale, float *out)
{
    for (int o = 32; o > 0; o >>= 1) v += __shfl_down(v, o, 64);
    if ((threadIdx.x & 63) == 0) scratch[threadIdx.x >> 6] = v;
    __syncthreads();
    if (threadIdx.x == 0) {
        float t[NG];
#pragma unroll
        for (int i = 0; i < NG; ++i) t[i] = scratch[i];
#pragma unroll
        for (int w = NG / 2; w > 0; w >>= 1)
#pragma unroll
            for (int i = 0; i < w; ++i) t[i] += t[i + w];
        *out = scale * t[0];
    }
}

template <int R, int NTH, int OQ>
__global__ __launch_bounds__(NTH) __attribute__((amdgpu_waves_per_eu(4))) void adjoint_tile_kernel(
    const float *v_all, const float *u_all, const float *an_all, float *ac_all, float *ap_all,
    const uint8_t *__restrict__ mask_all, int H, int W, int nbx, int tiles_per_img, StepArgs a,
    float lam_scale, int kflags, float *lam_partials, int lam_stride)
{
    using G = AdjTileGeo<R, NTH, OQ>;
    constexpr int OF = G::OF, h = G::h;
    __shared__ __attribute__((aligned(16))) float smem[G::LDS];
    float *sE = smem, *sD = smem + G::NE, *sX = sD + G::ND, *sP = sX + G::NX;
    const int tile = __builtin_amdgcn_readfirstlane(xcd_tile(blockIdx.x, gridDim.x));
    const int bimg = tile / tiles_per_img, tl = tile - bimg * tiles_per_img;
    const int ty = tl / nbx, tx = tl - ty * nbx;
    const int tid = threadIdx.x, lane = tid & 63;
    const int grp = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int X0 = tx * G::SW, Y0 = ty * G::TH;
    if constexpr (kLdsSentinel) sentinel_fill_block(smem, G::LDS);

    // resources based at the lowest row a needed value comes from
    const unsigned W4 = 4u * (unsigned)W;
    const int b0 = Y0 - h > 0 ? Y0 - h : 0;
    const int nrow = G::QH + 2;
    const int nb = H - b0 < nrow ? H - b0 : nrow;
    const size_t base = (size_t)bimg * H * W + (size_t)b0 * W;
    const __amdgpu_buffer_rsrc_t rs_v = buffer_rsrc(v_all + base, (unsigned)nb * W4);
    const __amdgpu_buffer_rsrc_t rs_u = buffer_rsrc(u_all + base, (unsigned)nb * W4);
    const __amdgpu_buffer_rsrc_t rs_an = buffer_rsrc(an_all + base, (unsigned)nb * W4);
    const __amdgpu_buffer_rsrc_t rs_m = buffer_rsrc(mask_all + base, (unsigned)nb * (unsigned)W);
    const int first = kflags & 1, fresh = kflags & 2;
    const __amdgpu_buffer_rsrc_t rs_ac = buffer_rsrc(ac_all + base, (unsigned)nb * W4);
    // ubar^k as read: no records in a cycle's first reverse step, where it is 0
    const __amdgpu_buffer_rsrc_t rs_acl = buffer_rsrc(ac_all + base, fresh ? 0u : (unsigned)nb * W4);
    // at k = 0 the (1 - alpha) r term stays in ubar^k: stores to ubar^{k-1} are dropped
    const __amdgpu_buffer_rsrc_t rs_ap = buffer_rsrc(ap_all + base, first ? 0u : (unsigned)nb * W4);

    const int cl = X0 - G::hc + lane;
    const unsigned cm = (unsigned)mirror_index(cl, W);
    const bool out_lane = lane >= G::hc && lane < 64 - G::hc && cl < W;
    const unsigned vo4 = out_lane ? 4u * (unsigned)cl : kOffNone;
    const unsigned vo1 = out_lane ? (unsigned)cl : kOffNone;

    // ---- Q ----
    const int q0 = Y0 - (R + 1) + grp * OQ;                   // image row of the group's q row 0
    float v[OQ + 2], u[OQ + 2], r[OQ + 2];
    unsigned mk[OQ + 2];
    const bool tiny = H < nrow;                               // may need repeated reflection
#pragma unroll
    for (int t = 0; t < OQ + 2; ++t) {
        int y = tiny ? mirror_reflect(q0 - 1 + t, H) : mirror_once(q0 - 1 + t, H);
        y = y < b0 ? b0 : y;                                  // rows no needed value comes from
        const unsigned ro = uniform_row((y < b0 + nb ? y : b0 + nb - 1) - b0);
        v[t] = buf_f32(rs_v, 4u * cm, ro * W4);
        u[t] = buf_f32(rs_u, 4u * cm, ro * W4);
        r[t] = buf_f32(rs_an, 4u * cm, ro * W4);
        mk[t] = __builtin_amdgcn_raw_buffer_load_b8(rs_m, cm, ro * (unsigned)W, 0);
    }
    float il2 = a.inv_lam2;
    asm volatile("" : "+v"(il2));
    float du[OQ + 2], dr[OQ + 2];
#pragma unroll
    for (int t = 0; t < OQ + 2; ++t) {
        r[t] = mk[t] ? 0.0f : r[t];
        du[t] = from_next_lane(u[t]) - from_prev_lane(u[t]);
        dr[t] = from_next_lane(r[t]) - from_prev_lane(r[t]);
    }
    float txx[OQ], tyy[OQ], z[OQ], ex[OQ], qy[OQ], dsum = 0.0f;
#pragma unroll
    for (int t = 0; t < OQ; ++t) {
        const float gxs = from_next_lane(v[t + 1]) - from_prev_lane(v[t + 1]);   // 2 gx
        const float gys = v[t + 2] - v[t];                                       // 2 gy
        const float hxx = lane_diff2(lane_diff(u[t + 1]));
        const float hyy = (u[t + 2] - u[t + 1]) - (u[t + 1] - u[t]);
        const float hxy = 0.25f * (du[t + 2] - du[t]);
        const float axx = lane_diff2(lane_diff(r[t + 1]));
        const float ayy = (r[t + 2] - r[t + 1]) - (r[t + 1] - r[t]);
        const float axy = 0.25f * (dr[t + 2] - dr[t]);
        float txy, qx, sds;
        adjoint_point(0.5f * gxs, 0.5f * gys, il2, axx, ayy, axy, hxx, hyy, hxy, txx[t],
                           tyy[t], txy, qx, qy[t], sds);
        const int g = q0 + t;                                 // image row
        dsum += (g >= Y0 && g < Y0 + G::TH && g < H && out_lane) ? sds : 0.0f;
        z[t] = from_next_lane(txy) - from_prev_lane(txy);
        ex[t] = from_next_lane(qx) - from_prev_lane(qx);
    }
    float *e0 = sE + grp * 384 + lane;
    e0[0] = tyy[0];
    e0[64] = z[0];
    e0[128] = qy[0];
    e0[192] = tyy[OQ - 1];
    e0[256] = z[OQ - 1];
    e0[320] = qy[OQ - 1];
    // what the update of the group's output rows reads
    const int Yf = Y0 + grp * OF;
    float an[OF], ac[OF];
    unsigned om[OF];
#pragma unroll
    for (int j = 0; j < OF; ++j) {
        const int o = Yf + j < H ? Yf + j : H - 1;
        const unsigned ro = uniform_row((o < b0 + nb ? o : b0 + nb - 1) - b0);
        an[j] = buf_f32(rs_an, vo4, ro * W4);
        ac[j] = buf_f32(rs_acl, vo4, ro * W4);
        om[j] = __builtin_amdgcn_raw_buffer_load_b8(rs_m, vo1, ro * (unsigned)W, 0);
    }
    __syncthreads();

    // ---- D: rows above the group's first and below its last from its neighbours
    // (the outermost rows of the tile are not needed) ----
    {
        const float *eu = sE + (grp > 0 ? grp - 1 : 0) * 384 + lane;
        const float *ed = sE + (grp + 1 < G::NG ? grp + 1 : grp) * 384 + lane;
        const float tyu = eu[192], zu = eu[256], qu = eu[320], tyd = ed[0], zd = ed[64], qd = ed[128];
#pragma unroll
        for (int t = 0; t < OQ; ++t) {
            const float qn = t + 1 < OQ ? qy[t + 1 < OQ ? t + 1 : 0] : qd;
            const float qp = t > 0 ? qy[t > 0 ? t - 1 : 0] : qu;
            const int dr_ = grp * OQ + t - 1;                 // row of d
            if (dr_ >= 0 && dr_ < G::DH) sD[dr_ * G::DS + G::PL + lane] = adj_div(ex[t], qn - qp);
            const int o = dr_ - R;                            // output row
            if (o >= 0 && o < G::TH) {
                const float tn = t + 1 < OQ ? tyy[t + 1 < OQ ? t + 1 : 0] : tyd;
                const float tp = t > 0 ? tyy[t > 0 ? t - 1 : 0] : tyu;
                const float zn = t + 1 < OQ ? z[t + 1 < OQ ? t + 1 : 0] : zd;
                const float zp = t > 0 ? z[t > 0 ? t - 1 : 0] : zu;
                sP[o * 64 + lane] = adj_outer(lane_diff2(lane_diff(txx[t])),
                                              (tn - tyy[t]) - (tyy[t] - tp), zn, zp);
            }
        }
    }
    float wv[2 * R + 1], alpha = a.alpha, tau = a.tau, keep_back = first ? 1.0f : 0.0f;
    vector_weights<R>(a.w, wv);
    asm volatile("" : "+v"(alpha), "+v"(tau), "+v"(keep_back));
    __syncthreads();

    // ---- X ----
#pragma unroll
    for (int k = 0; k < (G::DH * G::NQ + NTH - 1) / NTH; ++k) {
        const int it = tid + k * NTH;
        if (it < G::DH * G::NQ) {
            const int row = it / G::NQ, q = it - row * G::NQ + G::Q0;
            const f32x4 *src = reinterpret_cast<const f32x4 *>(sD + row * G::DS + G::PL + 4 * (q - G::C4));
            float win[4 * G::NF4];
#pragma unroll
            for (int f = 0; f < G::NF4; ++f) {
                const f32x4 x = src[f];
#pragma unroll
                for (int e = 0; e < 4; ++e) win[4 * f + e] = x[e];
            }
            f32x4 o;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                float acc = wv[0] * win[G::OFF + e];
#pragma unroll
                for (int j = 1; j <= 2 * R; ++j) acc = fmaf(wv[j], win[G::OFF + e + j], acc);
                o[e] = acc;
            }
            *reinterpret_cast<f32x4 *>(sX + 64 * row + 4 * q) = o;
        }
    }
    __syncthreads();

    // ---- F ----
    if (Yf < H) {
        const float *px = sX + 64 * (grp * OF) + lane, *pp = sP + 64 * (grp * OF) + lane;
#pragma unroll
        for (int j = 0; j < OF; ++j) {
            if (grp * OF + j >= G::TH || Yf + j >= H) break;  // (wave-uniform)
            float cq = 0.0f;
#pragma unroll
            for (int t = 0; t <= 2 * R; ++t) cq = fmaf(wv[t], px[64 * (j + t)], cq);
            float back;
            const float acv = adj_update(pp[64 * j], cq, an[j], ac[j], om[j] != 0, tau, alpha,
                                         keep_back, back);
            const unsigned ro = (unsigned)(Yf + j - b0) * W4;
            __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(back), rs_ap, vo4, ro, 0);
            __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(acv), rs_ac, vo4, ro, 0);
        }
    }
    group_sum<G::NG>(dsum, sE, lam_scale, lam_partials + (size_t)bimg * lam_stride + tl);
}

// ---- fused reverse step on wave strips ----
//
// A wave owns 64 consecutive columns c = X0-2-R .. X0+61-R (one per lane) and
// streams down the rows of a segment.  For each stream row i it loads the
// presmoothed image v = K_sigma * u^k (kept by the forward recompute), u^k and
// r = mbar ubar^{k+1} of the row, then
//   S3  at row g = i-1: gradient of v, Hessians of u and of r (the last three
//       rows in registers, lane neighbours by DPP) and the adjoint point
//       quantities D:A, q, de/dlambda;
//   S4  at row g-1: P(u) r from the outer differences of D:A, and
//       d = -div q, whose x pass goes through a one-row LDS buffer into a
//       register window;
//   S5  at row o = i-R-2: y pass of d (C^T q) and the reverse update.
// Lanes R+2 .. 61-R own output columns (60-2R per wave).  The input halo is
// R+2 rows each way: R+1 for the y pass of d and one more for q.
template <int R, int ROWS>
struct AdjStripGeo {
    static constexpr int P = 2 * R + 1;                       // d window length
    static constexpr int U = P;                               // unroll (window slots constant)
    static constexpr int h = R + 2;                           // input row halo
    static constexpr int hc = R + 2;                          // first output lane
    static constexpr int SW = 64 - 2 * hc;                    // output columns per wave
    static constexpr int ND = 64 + 2 * R;                     // d row, R pad on each side
    static constexpr int M = (ROWS + 2 * h + U - 1) / U;      // main-loop iterations
    static constexpr int NROW = M * U;                        // rows streamed per wave
    static constexpr int OH = NROW - 2 * h;                   // output rows per wave
    static constexpr int LDS = ND + P * 64;                   // floats of LDS per wave
    static_assert(rows_addressable(NROW), "row offsets");
};

struct AdjStripArgs {
    const float *v, *u, *an;    // K_sigma * u^k, u^k, ubar^{k+1}
    float *ac, *ap;             // ubar^k (accumulated in place), ubar^{k-1} contribution
    const uint8_t *mask;
    int H, W, X0, Y0;
    float tau, alpha, il2;      // il2 = 1/lambda^2
    int first;                  // k == 0: the (1-alpha) r term goes to ubar^k itself
    int fresh;                  // k == n-1: ubar^k starts at 0 (not read)
    int model;                  // tensor variant (GEN kernels only)
    int prio;                   // lower the issue priority along the segment
};

// Global loads of one stream row: v, u^k and r of the row itself, and
// ubar^{k+1}, ubar^k and the mask of the output row it serves.
struct AdjStripRow {
    float v, u, rn, oa, oc;
    unsigned rmk, omk;
};

template <int R, int ROWS, bool GEN = false>
__device__ __forceinline__ void adjoint_strip_step(float *lds, const AdjStripArgs &s,
                                                   const float (&w)[2 * kRMax + 1],
                                                   float *partial, float lam_scale)
{
    using G = AdjStripGeo<R, ROWS>;
    constexpr int P = G::P, U = G::U, h = G::h;
    const int lane = threadIdx.x & 63;
    const int H = s.H, W = s.W;
    const unsigned W4 = 4u * (unsigned)W;
    if constexpr (kLdsSentinel) sentinel_fill_wave(lds, G::LDS);

    // resources based at the lowest row a needed value comes from (as in
    // the forward strip)
    const int ybase = s.Y0 - h;                               // image row of stream row 0
    const int b0 = ybase > 0 ? ybase : 0;
    const int nb = (H - b0 < G::NROW) ? H - b0 : G::NROW;
    const size_t base = (size_t)b0 * W;
    const __amdgpu_buffer_rsrc_t rs_v = buffer_rsrc(s.v + base, (unsigned)nb * W4);
    const __amdgpu_buffer_rsrc_t rs_u = buffer_rsrc(s.u + base, (unsigned)nb * W4);
    const __amdgpu_buffer_rsrc_t rs_an = buffer_rsrc(s.an + base, (unsigned)nb * W4);
    const __amdgpu_buffer_rsrc_t rs_ac = buffer_rsrc(s.ac + base, (unsigned)nb * W4);
    // ubar^k as read: no records in a cycle's first reverse step, where it
    // starts at 0 (its loads then read 0, and no clearing pass is needed)
    const __amdgpu_buffer_rsrc_t rs_acl = buffer_rsrc(s.ac + base, s.fresh ? 0u : (unsigned)nb * W4);
    // at k = 0 the (1 - alpha) r term stays in ubar^k: the ubar^{k-1} resource
    // then has no records, so its stores are dropped
    const __amdgpu_buffer_rsrc_t rs_ap = buffer_rsrc(s.ap + base, s.first ? 0u : (unsigned)nb * W4);
    const float keep_back = s.first ? 1.0f : 0.0f;
    const __amdgpu_buffer_rsrc_t rs_m = buffer_rsrc(s.mask + base, (unsigned)nb * (unsigned)W);

    const int cl = s.X0 - G::hc + lane;                       // this lane's column
    const unsigned cm = (unsigned)mirror_reflect(cl, W);      // ... mirrored into the image
    const bool out_lane = lane >= G::hc && lane < 64 - G::hc && cl < W;
    const unsigned vo4 = out_lane ? 4u * (unsigned)cl : kOffNone;
    const unsigned vo1 = out_lane ? (unsigned)cl : kOffNone;
    const int yend = s.Y0 + G::OH < H ? s.Y0 + G::OH : H;     // rows owned: [Y0, yend)

    // the d row (lane l at l + R), then P(u) r of the last P rows (slot j,
    // lane l at j * 64 + l): a slot is read R rows after it is written, and a
    // register window would cost more VGPRs than its P values
    float *dw = lds + lane;
    float *prr = lds + G::ND + lane;

    float wv[2 * R + 1];
    if constexpr (!GEN) {
        vector_weights<R>(w, wv);
    } else {                          // the variants have no registers left at 4 waves a SIMD
#pragma unroll
        for (int j = 0; j <= 2 * R; ++j) wv[j] = w[j];
    }
    float dwin[P];                    // x-pass d; stream row j in slot j % P
#pragma unroll
    for (int j = 0; j < P; ++j) dwin[j] = 0.0f;
    float v_m1 = 0.0f, v_m2 = 0.0f;                          // v at rows g, g-1
    // u and r at row g, their differences to row g-1, and along x their first (row g)
    // and central (rows g, g-1) differences, taken when a row arrives
    float u_m1 = 0.0f, eu_m1 = 0.0f, fu_m1 = 0.0f, du_m1 = 0.0f, du_m2 = 0.0f;
    float r_m1 = 0.0f, er_m1 = 0.0f, fr_m1 = 0.0f, dr_m1 = 0.0f, dr_m2 = 0.0f;
    // (D:A)xx: x difference at row g-1; (D:A)yy at row g-1, and less row g-2
    float ftx_p = 0.0f, tyy_p = 0.0f, ety_p = 0.0f;
    float z_p = 0.0f, z_pp = 0.0f;                           // (D:A)xy(l+1)-(D:A)xy(l-1)
    float qx_p = 0.0f, qy_p = 0.0f, qy_pp = 0.0f;            // q at rows g-1 (g-2 for y)
    float dsum = 0.0f;                                       // de/dlambda over the lane's rows

    RowTrack ty;                      // next prefetch: its mirrored image row
    ty.init(ybase, H);
    int on = ybase - h;                                       // output row it serves
    // ubar^{k+1} and the mask at output row o are those the stream read at its
    // row o, h rows earlier (same column on output lanes, no mirroring inside
    // the image).  Where the unrolled row block covers h + 1 rows (R >= 2) they
    // are kept in registers indexed by stream row % U instead of being loaded
    // again: by then the rows have left L2 (about 5 of the 22 bytes a pixel
    // otherwise fetches).
    constexpr bool OREG = U >= h + 1;
    constexpr int OQ = OREG ? U : 1;
    float rnq[OQ];
    unsigned rmq[OQ];
#pragma unroll
    for (int j = 0; j < OQ; ++j) {
        rnq[j] = 0.0f;
        rmq[j] = 0u;
    }
    auto prefetch = [&](AdjStripRow &r) {
        const unsigned sr = (unsigned)((ty.y > b0 ? ty.y : b0) - b0);
        r.v = buf_f32(rs_v, 4u * cm, sr * W4);
        r.u = buf_f32(rs_u, 4u * cm, sr * W4);
        r.rn = buf_f32(rs_an, 4u * cm, sr * W4);
        r.rmk = __builtin_amdgcn_raw_buffer_load_b8(rs_m, cm, sr * (unsigned)W, 0);
        int oc = on < b0 ? b0 : on;                           // clamped; unused rows are not stored
        oc = oc > H - 1 ? H - 1 : oc;
        const unsigned ro = (unsigned)(oc - b0);
        if constexpr (!OREG) {
            r.oa = buf_f32(rs_an, vo4, ro * W4);
            r.omk = __builtin_amdgcn_raw_buffer_load_b8(rs_m, vo1, ro * (unsigned)W, 0);
        }
        r.oc = buf_f32(rs_acl, vo4, ro * W4);
        ty.next(H);
        ++on;
    };
    AdjStripRow r0, r1;
    r0.oa = r1.oa = 0.0f;
    r0.omk = r1.omk = 0u;
    prefetch(r0);
    prefetch(r1);

#pragma unroll 1
    for (int it = 0; it < G::M; ++it) {
        // With every wave of the launch resident at once, waves further down
        // their segment yield issue slots to those behind, as in the forward
        // strip; when the launch needs more than one round of waves the host
        // leaves this off (late waves would then hold the top priority).  Only
        // the short segments, which small problems use, carry the code.  The
        // levels stay above 0, the level of the recompute steps that run beside
        // this kernel on the other stream, so these waves, the critical path,
        // issue first.
        if (ROWS <= 28 && s.prio) {
            const int left = G::M - it;
            if (left >= 3) __builtin_amdgcn_s_setprio(3);
            else if (left == 2) __builtin_amdgcn_s_setprio(2);
            else __builtin_amdgcn_s_setprio(1);
        }
#pragma unroll
        for (int ph = 0; ph < U; ++ph) {
            const int i = it * U + ph;                        // stream row (wave-uniform)
            const AdjStripRow cur = r0;
            r0 = r1;
            prefetch(r1);
            if constexpr (OREG) {
                rnq[ph] = cur.rn;                                    // stream row i % U = ph
                rmq[ph] = cur.rmk;
            }

            // ---- S3 at row g = i - 1 (rows g-1, g, g+1: m2, m1, this row) ----
            const float v_p1 = cur.v, u_p1 = cur.u;
            const float r_p1 = cur.rmk ? 0.0f : cur.rn;
            const float gxs = from_next_lane(v_m1) - from_prev_lane(v_m1);  // 2 gx
            const float gys = v_p1 - v_m2;                                   // 2 gy
            const float du_p1 = from_next_lane(u_p1) - from_prev_lane(u_p1);  // row g+1
            const float dr_p1 = from_next_lane(r_p1) - from_prev_lane(r_p1);
            const float eu_p1 = u_p1 - u_m1, er_p1 = r_p1 - r_m1;
            const float hxx = lane_diff2(fu_m1), axx = lane_diff2(fr_m1);
            const float hyy = eu_p1 - eu_m1, ayy = er_p1 - er_m1;
            const float hxy = 0.25f * (du_p1 - du_m2);
            const float axy = 0.25f * (dr_p1 - dr_m2);
            v_m2 = v_m1;
            v_m1 = v_p1;
            u_m1 = u_p1;
            eu_m1 = eu_p1;
            fu_m1 = lane_diff(u_p1);
            r_m1 = r_p1;
            er_m1 = er_p1;
            fr_m1 = lane_diff(r_p1);
            du_m2 = du_m1;
            du_m1 = du_p1;
            dr_m2 = dr_m1;
            dr_m1 = dr_p1;
            float tx, ty_, txy, qx, qy, sds;
            adjoint_point<GEN>(0.5f * gxs, 0.5f * gys, s.il2, axx, ayy, axy, hxx, hyy, hxy, tx, ty_,
                               txy, qx, qy, sds, s.model);
            const int g = ybase + i - 1;                              // image row of S3
            dsum += (g >= s.Y0 && g < yend && out_lane) ? sds : 0.0f;
            const float z = from_next_lane(txy) - from_prev_lane(txy);

            // ---- S4 at row g - 1: P(u) r and d = -div q ----
            const float ety = ty_ - tyy_p;
            const float pr = adj_outer(lane_diff2(ftx_p), ety - ety_p, z, z_pp);
            const float d = adj_div(from_next_lane(qx_p) - from_prev_lane(qx_p), qy - qy_pp);
            dw[R] = d;
            wave_lds_sync();
            float dx = wv[0] * dw[0];
#pragma unroll
            for (int j = 1; j <= 2 * R; ++j) dx = fmaf(wv[j], dw[j], dx);
            const int jd = ((ph - 2) % P + P) % P;                    // slot of stream row i - 2
            dwin[jd] = dx;
            prr[jd * 64] = pr;
            ety_p = ety;
            tyy_p = ty_;
            ftx_p = lane_diff(tx);
            z_pp = z_p;
            z_p = z;
            qy_pp = qy_p;
            qy_p = qy;
            qx_p = qx;

            // ---- S5: output row o (stream row i - h) ----
            const int o = ybase + i - h;
            if (i >= 2 * h && o < H) {
                float cq = 0.0f;                                     // stream rows i-h-R .. i-2
#pragma unroll
                for (int j = 0; j <= 2 * R; ++j)
                    cq = fmaf(wv[j], dwin[((ph - h - R + j) % P + P) % P], cq);
                const float pro = prr[((ph - h) % P + P) % P * 64];
                const int so = ((ph - h) % U + U) % U;              // stream row i - h
                const float anv = OREG ? rnq[so] : cur.oa;
                const bool mk = (OREG ? rmq[so] : cur.omk) != 0;
                float back;
                const float acv = adj_update(pro, cq, anv, cur.oc, mk, s.tau, s.alpha, keep_back,
                                             back);
                const unsigned ro = (unsigned)(o - b0) * W4;
                __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(back), rs_ap, vo4, ro, 0);
                __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(acv), rs_ac, vo4, ro, 0);
            }
        }
    }
    // pairwise tree over the lanes; every lane stores lane 0's total (no
    // lane-dependent branch)
    for (int off = 32; off > 0; off >>= 1) dsum += __shfl_down(dsum, off, 64);
    const float tot = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(dsum), 0));
    partial[0] = lam_scale * tot;
}

template <int R, int ROWS, bool GEN>
__device__ __forceinline__ void adjoint_strip_body(const float *v_all, const float *u_all,
                                                   const float *an_all,
                                                   float *ac_all, float *ap_all,
                                                   const uint8_t *__restrict__ mask_all, int H,
                                                   int W, int nstrip, int per_img, int nitems,
                                                   const StepArgs &a, float lam_scale,
                                                   int kflags, int prio, float *lam_partials,
                                                   int lam_stride)
{
    using G = AdjStripGeo<R, ROWS>;
    __shared__ float lds[4 * G::LDS];
    const int wave = threadIdx.x >> 6;
    const int item = __builtin_amdgcn_readfirstlane(xcd_tile(blockIdx.x, gridDim.x) * 4 + wave);
    if (item >= nitems) return;  // whole wave; the kernel has no workgroup barrier
    const int b = item / per_img;
    const int r = item - b * per_img;
    const int seg = r / nstrip, strip = r - seg * nstrip;
    const size_t off = (size_t)b * H * W;
    AdjStripArgs s;
    s.v = v_all + off;
    s.u = u_all + off;
    s.an = an_all + off;
    s.ac = ac_all + off;
    s.ap = ap_all + off;
    s.mask = mask_all + off;
    s.H = H;
    s.W = W;
    s.X0 = strip * G::SW;
    s.Y0 = seg * G::OH;
    s.tau = a.tau;
    s.alpha = a.alpha;
    s.il2 = a.inv_lam2;
    s.first = kflags & 1;
    s.fresh = (kflags >> 1) & 1;
    s.model = a.model;
    s.prio = prio;
    adjoint_strip_step<R, ROWS, GEN>(lds + wave * G::LDS, s, a.w,
                                     lam_partials + (size_t)b * lam_stride + r, lam_scale);
}

template <int R, int ROWS>
__global__ __launch_bounds__(256) void adjoint_strip_kernel(const float *v_all, const float *u_all,
                                                            const float *an_all,
                                                            float *ac_all, float *ap_all,
                                                            const uint8_t *__restrict__ mask_all,
                                                            int H, int W, int nstrip, int per_img,
                                                            int nitems, StepArgs a,
                                                            float lam_scale, int kflags,
                                                            int prio, float *lam_partials,
                                                            int lam_stride)
{
    adjoint_strip_body<R, ROWS, false>(v_all, u_all, an_all, ac_all, ap_all, mask_all, H, W, nstrip,
                                       per_img, nitems, a, lam_scale, kflags, prio,
                                       lam_partials, lam_stride);
}

// The reverse step of the tensor variants (diffusivities of Table 7, mu3
// choices of Sec. 3.1) on strips of >= 28 rows.
template <int R>
__global__ __launch_bounds__(256) void adjoint_strip_model_kernel(
    const float *v_all, const float *u_all, const float *an_all, float *ac_all, float *ap_all,
    const uint8_t *__restrict__ mask_all, int H, int W, int nstrip, int per_img, int nitems,
    StepArgs a, float lam_scale, int kflags, int prio, float *lam_partials,
    int lam_stride)
{
    adjoint_strip_body<R, 28, true>(v_all, u_all, an_all, ac_all, ap_all, mask_all, H, W, nstrip,
                                    per_img, nitems, a, lam_scale, kflags, prio, lam_partials,
                                    lam_stride);
}

// ---- small helper kernels ----
__global__ __launch_bounds__(256) void fill_kernel(float *p, size_t n, float v)
{
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (size_t)gridDim.x * blockDim.x)
        p[i] = v;
}

// One pass of the pairwise lambda reduction: out[b][c] = the sum of the c-th
// run of 2048 values of image b's row of in (length L, zero-padded), by a
// pairwise tree in LDS.  Passes repeat until one value per image remains.
__global__ __launch_bounds__(1024) void pairwise_pass_kernel(const float *in, long long L,
                                                             float *out, int nout)
{
    __shared__ float sv[2048];
    const int c = blockIdx.x, b = blockIdx.y, tid = threadIdx.x;
    const float *p = in + (size_t)b * L + (size_t)c * 2048;
    const long long lim = L - (long long)c * 2048;
    sv[tid] = tid < lim ? p[tid] : 0.0f;
    sv[tid + 1024] = tid + 1024 < lim ? p[tid + 1024] : 0.0f;
    __syncthreads();
    for (int s = 1024; s > 0; s >>= 1) {
        if (tid < s) sv[tid] = sv[tid] + sv[tid + s];
        __syncthreads();
    }
    if (tid == 0) out[(size_t)b * nout + c] = sv[0];
}

// Cascade of the per-cycle sums over cycles (a pairwise tree built like a
// binary counter): slot i holds the sum of a block of 2^i cycles.  Adding the
// j-th cycle sum merges it with the t = (trailing ones of j) lowest slots and
// stores the block in slot t.
__device__ __forceinline__ void lambda_carry(float v, float *slots, int B, int b, int t)
{
    for (int i = 0; i < t; ++i) v = slots[(size_t)i * B + b] + v;
    slots[(size_t)t * B + b] = v;
}

__global__ void lambda_carry_kernel(const float *cyc, float *slots, int B, int t)
{
    const int b = blockIdx.x * blockDim.x + threadIdx.x;
    if (b >= B) return;
    lambda_carry(cyc[b], slots, B, b, t);
}

// Both of the above in one launch when a cycle's partials fit one pairwise
// pass (L <= 2048 per image): the same tree and the same cascade, so the same
// bits, with one launch per cycle instead of two.
__global__ __launch_bounds__(1024) void lambda_cycle_kernel(const float *in, long long L,
                                                            float *slots, int b0, int B, int t)
{
    __shared__ float sv[2048];
    const int b = b0 + blockIdx.x, tid = threadIdx.x;
    const float *p = in + (size_t)b * L;
    sv[tid] = tid < L ? p[tid] : 0.0f;
    sv[tid + 1024] = tid + 1024 < L ? p[tid + 1024] : 0.0f;
    __syncthreads();
    for (int s = 1024; s > 0; s >>= 1) {
        if (tid < s) sv[tid] = sv[tid] + sv[tid + s];
        __syncthreads();
    }
    if (tid == 0) lambda_carry(sv[0], slots, B, b, t);
}

// dL/dlambda = the occupied slots (the set bits of the cycle count M), largest
// block first.
__global__ void lambda_final_kernel(const float *slots, int B, unsigned M, float *out)
{
    const int b = blockIdx.x * blockDim.x + threadIdx.x;
    if (b >= B) return;
    float v = 0.0f;
    bool any = false;
    for (int i = 31; i >= 0; --i)
        if ((M >> i) & 1u) {
            const float x = slots[(size_t)i * B + b];
            v = any ? v + x : x;
            any = true;
        }
    out[b] = v;
}

// On known pixels abar0 holds the sum of ubar over every state (ubar^{0,0}
// included): that is dL/df.  Elsewhere abar0 = ubar^{0,0} = dL/du_init.
__global__ __launch_bounds__(256) void adjoint_final_kernel(const float *abar0,
                                                            const uint8_t *__restrict__ mask,
                                                            float *gk, float *gi, size_t n)
{
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (size_t)gridDim.x * blockDim.x) {
        const float v = abar0[i];
        const bool m = mask[i] != 0;
        gk[i] = m ? v : 0.0f;
        gi[i] = m ? 0.0f : v;
    }
}

static unsigned grid_for(size_t n)
{
    size_t b = (n + 255) / 256;
    return (unsigned)(b > 8192 ? 8192 : (b < 1 ? 1 : b));
}

// Reverse tile of a forward tile shape: threads and q rows per group.
#define EED4_ADJ_TILES(CALL)                                          \
    case 0: return CALL(512, 6);                                      \
    case 1: return CALL(256, 6);                                      \
    default: return CALL(512, 4);

template <int R, int NTH, int OQ>
static int adj_tile_items_t(int H, int W)
{
    using G = AdjTileGeo<R, NTH, OQ>;
    return ((W + G::SW - 1) / G::SW) * ((H + G::TH - 1) / G::TH);
}

template <int R, int ROWS>
static int adj_strip_items_t(int H, int W)
{
    using G = AdjStripGeo<R, ROWS>;
    return ((W + G::SW - 1) / G::SW) * ((H + G::OH - 1) / G::OH);
}

// Segment heights of the strip reverse step per forward strip shape.  The
// shapes 3 and 7 map to segments of >= 80 rows: at 4096^2 and R = 6 those
// launch 4,042 waves, which all fit at once at 4 waves per SIMD (>= 64 rows
// launch 4,730, and the last 16 % ran as a second, nearly empty round).
template <int R>
static int adj_items_r(int shape, int H, int W)
{
    switch (shape) {
    case kShapeStrip:
    case kShapeStripWide: return adj_strip_items_t<R, 80>(H, W);
    case kShapeStripTall: return adj_strip_items_t<R, 136>(H, W);
    case kShapeStripShort:
    case kShapeStripWideShort: return adj_strip_items_t<R, 28>(H, W);
    case kShapeStripTiny: return adj_strip_items_t<R, 8>(H, W);
#define EED4_CALL_T(nth, oq) adj_tile_items_t<R, nth, oq>(H, W)
    EED4_ADJ_TILES(EED4_CALL_T)
#undef EED4_CALL_T
    }
}

#define EED4_RSWITCH(CALL)                                                          \
    switch (R) {                                                                    \
    case 0: return CALL(0); case 1: return CALL(1); case 2: return CALL(2);         \
    case 3: return CALL(3); case 4: return CALL(4); case 5: return CALL(5);         \
    case 6: return CALL(6); case 7: return CALL(7); case 8: return CALL(8);         \
    default: break;                                                                 \
    }

// Work items per image of a reverse step: tiles or strip segments.
static int adjoint_items(int R, int shape, int H, int W)
{
#define EED4_CALL_N(r) adj_items_r<r>(shape, H, W)
    EED4_RSWITCH(EED4_CALL_N)
#undef EED4_CALL_N
    return 0;
}

static int max_adjoint_items(int R, int H, int W)
{
    int m = 0;
    for (int sh = 0; sh < kNumShapes; ++sh) m = std::max(m, adjoint_items(R, sh, H, W));
    return m;
}

// Buffers of one reverse step.
struct RevStep {
    const float *v;          // K_sigma * u^k
    const float *u, *an;     // u^k, ubar^{k+1}
    float *ac, *ap;          // ubar^k (in place), ubar^{k-1} contribution
    const uint8_t *mask;
    float *lp;               // lambda partials of this step: image b, item r at lp[b * ls + r]
    int ls;                  // ... image stride (cycle_len * items per image)
    int B, H, W, R, shape, first;
    int fresh;               // a cycle's first reverse step: ubar^k starts at 0 (not read)
    int kflags() const { return (first ? 1 : 0) | (fresh ? 2 : 0); }
    // the step of images b0 .. b0 + n - 1 alone
    RevStep images(int b0, int n) const
    {
        const size_t o = (size_t)b0 * H * W;
        RevStep q = *this;
        q.v += o;
        q.u += o;
        q.an += o;
        q.ac += o;
        q.ap += o;
        q.mask += o;
        q.lp += (size_t)b0 * ls;
        q.B = n;
        return q;
    }
};

template <int R, int NTH, int OQ>
static hipError_t launch_rev_tile(const RevStep &t, const StepArgs &a, float ls, hipStream_t s)
{
    using G = AdjTileGeo<R, NTH, OQ>;
    const int nbx = (t.W + G::SW - 1) / G::SW;
    const int tpi = adj_tile_items_t<R, NTH, OQ>(t.H, t.W);
    return launch_batches(t.B, tpi, 1, NTH, [&](int b0, int n, unsigned blocks) {
        const RevStep q = t.images(b0, n);
        hipLaunchKernelGGL((adjoint_tile_kernel<R, NTH, OQ>), dim3(blocks), dim3(NTH), 0, s, q.v, q.u,
                           q.an, q.ac, q.ap, q.mask, q.H, q.W, nbx, tpi, a, ls, q.kflags(), q.lp,
                           q.ls);
    });
}

// Waves of kernel k (256-thread workgroups) the current device holds at once;
// 0 if the runtime cannot tell.  The launchers keep the first answer (the
// devices of one node are alike); a wrong answer only switches the issue
// priority schedule on or off, never the results.
template <typename K>
static long long resident_waves(K k)
{
    int per_cu = 0, dev = 0, cus = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, k, 256, 0) != hipSuccess) return 0;
    if (hipGetDevice(&dev) != hipSuccess) return 0;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess)
        return 0;
    return 4LL * per_cu * cus;
}

template <int R, int ROWS>
static hipError_t launch_rev_strip(const RevStep &t, const StepArgs &a, float ls,
                                   hipStream_t s)
{
    using G = AdjStripGeo<R, ROWS>;
    const int nstrip = (t.W + G::SW - 1) / G::SW;
    const int per_img = adj_strip_items_t<R, ROWS>(t.H, t.W);
    // the issue-priority schedule only when every wave is resident at once
    static const long long cap = resident_waves(adjoint_strip_kernel<R, ROWS>);
    const int prio = (long long)per_img * t.B <= cap ? 1 : 0;
    return launch_batches(t.B, per_img, 4, 256, [&](int b0, int n, unsigned blocks) {
        const RevStep q = t.images(b0, n);
        hipLaunchKernelGGL((adjoint_strip_kernel<R, ROWS>), dim3(blocks), dim3(256), 0, s, q.v, q.u,
                           q.an, q.ac, q.ap, q.mask, q.H, q.W, nstrip, per_img, per_img * n, a, ls,
                           q.kflags(), prio, q.lp, q.ls);
    });
}

template <int R>
static hipError_t launch_rev_model(const RevStep &t, const StepArgs &a, float ls,
                                   hipStream_t s)
{
    using G = AdjStripGeo<R, 28>;
    const int nstrip = (t.W + G::SW - 1) / G::SW;
    const int per_img = adj_strip_items_t<R, 28>(t.H, t.W);
    static const long long cap = resident_waves(adjoint_strip_model_kernel<R>);
    const int prio = (long long)per_img * t.B <= cap ? 1 : 0;
    return launch_batches(t.B, per_img, 4, 256, [&](int b0, int n, unsigned blocks) {
        const RevStep q = t.images(b0, n);
        hipLaunchKernelGGL((adjoint_strip_model_kernel<R>), dim3(blocks), dim3(256), 0, s, q.v, q.u,
                           q.an, q.ac, q.ap, q.mask, q.H, q.W, nstrip, per_img, per_img * n, a, ls,
                           q.kflags(), prio, q.lp, q.ls);
    });
}

template <int R>
static hipError_t launch_rev_r(const RevStep &t, const StepArgs &a, float ls,
                               hipStream_t s)
{
    // tensor variants: one kernel shape (strips of >= 28 rows)
    if (a.model != 0)
        return t.shape == kShapeStripShort ? launch_rev_model<R>(t, a, ls, s)
                                           : hipErrorInvalidValue;
    switch (t.shape) {
    case kShapeStrip:
    case kShapeStripWide: return launch_rev_strip<R, 80>(t, a, ls, s);
    case kShapeStripTall: return launch_rev_strip<R, 136>(t, a, ls, s);
    case kShapeStripShort:
    case kShapeStripWideShort: return launch_rev_strip<R, 28>(t, a, ls, s);
    case kShapeStripTiny: return launch_rev_strip<R, 8>(t, a, ls, s);
#define EED4_CALL_T(nth, oq) launch_rev_tile<R, nth, oq>(t, a, ls, s)
    EED4_ADJ_TILES(EED4_CALL_T)
#undef EED4_CALL_T
    }
}

// One reverse step k (alpha_k; the pixels' s de/ds sum to dL/dlambda with the
// scale alpha_k tau / lambda).
static hipError_t launch_reverse_step(const RevStep &t, const eed4_params *p, int k,
                                      hipStream_t s)
{
    const StepArgs a = make_args(p->sigma, t.R, p->tau, p->lambda, k, model_of_flags(p->flags));
    const float ls = (float)((double)a.alpha * a.tau / p->lambda);
    const int R = t.R;
#define EED4_CALL_REV(r) launch_rev_r<r>(t, a, ls, s)
    EED4_RSWITCH(EED4_CALL_REV)
#undef EED4_CALL_REV
    return hipErrorInvalidValue;
}
#undef EED4_RSWITCH

static hipError_t launch_fill(float *p, size_t n, float v, hipStream_t s)
{
    hipLaunchKernelGGL(fill_kernel, dim3(grid_for(n)), dim3(256), 0, s, p, n, v);
    return hipGetLastError();
}

// Pairwise sum of each image's row of L values (in[b * L + i]) into out[b],
// through tmp1 / tmp2 (B * ceil(L / 2048) and B * ceil(L / 2048^2) floats).
static hipError_t launch_pairwise_sum(const float *in, long long L, int B, float *tmp1,
                                      float *tmp2, float *out, hipStream_t s)
{
    const float *src = in;
    float *bufs[2] = {tmp1, tmp2};
    int which = 0;
    for (;;) {
        const long long nout = (L + 2047) / 2048;
        float *dst = nout == 1 ? out : bufs[which];
        hipLaunchKernelGGL(pairwise_pass_kernel, dim3((unsigned)nout, (unsigned)B), dim3(1024), 0,
                           s, src, L, dst, (int)nout);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess || nout == 1) return e;
        src = dst;
        L = nout;
        which ^= 1;
    }
}

static hipError_t launch_lambda_carry(const float *cyc, float *slots, int B, int t, hipStream_t s)
{
    hipLaunchKernelGGL(lambda_carry_kernel, dim3((B + 255) / 256), dim3(256), 0, s, cyc, slots, B,
                       t);
    return hipGetLastError();
}

static hipError_t launch_lambda_final(const float *slots, int B, int M, float *out, hipStream_t s)
{
    hipLaunchKernelGGL(lambda_final_kernel, dim3((B + 255) / 256), dim3(256), 0, s, slots, B,
                       (unsigned)M, out);
    return hipGetLastError();
}

static hipError_t launch_adjoint_final(const float *abar0, const uint8_t *mask, float *gk,
                                       float *gi, size_t n, hipStream_t s)
{
    hipLaunchKernelGGL(adjoint_final_kernel, dim3(grid_for(n)), dim3(256), 0, s, abar0, mask, gk,
                       gi, n);
    return hipGetLastError();
}

// ---- workspace layout of eed4_backward ----
struct BackwardLayout {
    size_t U, V, an, ac, ap, lp, t1, t2, cyc, slots, total;
};

static BackwardLayout backward_layout(int B, int H, int W, int n, int R)
{
    BackwardLayout L{};
    const size_t N = (size_t)B * H * W;
    size_t o = 0;
    // two sets of recompute buffers: cycle m-1 is recomputed while cycle m is reversed
    L.U = o; o = align_up(o + sizeof(float) * N * 2 * (size_t)(n > 1 ? n - 1 : 1));
    // ... and K_sigma * u^{m,k}, k = 0 .. n-1, for the reverse step
    L.V = o; o = align_up(o + sizeof(float) * N * 2 * (size_t)(n > 0 ? n : 1));
    L.an = o; o = align_up(o + sizeof(float) * N);
    L.ac = o; o = align_up(o + sizeof(float) * N);
    L.ap = o; o = align_up(o + sizeof(float) * N);
    // lambda: one FP32 partial per work item and reverse step of a cycle, the
    // pairwise passes over them, the cycle sum and 32 cascade slots (per image)
    const size_t per_img = (size_t)(n > 0 ? n : 1) * (size_t)max_adjoint_items(R, H, W);
    const size_t n1 = (per_img + 2047) / 2048, n2 = (n1 + 2047) / 2048;
    L.lp = o; o = align_up(o + sizeof(float) * per_img * B);
    L.t1 = o; o = align_up(o + sizeof(float) * n1 * B);
    L.t2 = o; o = align_up(o + sizeof(float) * n2 * B);
    L.cyc = o; o = align_up(o + sizeof(float) * (size_t)B);
    L.slots = o; o = align_up(o + sizeof(float) * 32 * (size_t)B);
    L.total = o;
    return L;
}

size_t backward_workspace(int B, int H, int W, const eed4_params *p)
{
    const int R = eed4_radius(p->sigma);
    return R < 0 ? 0 : backward_layout(B, H, W, p->cycle_len, R).total;
}

static std::string adjoint_tune_key(int R, int B, int H, int W)
{
    char buf[96];
    std::snprintf(buf, sizeof(buf), "adjoint_R%d_B%d_H%d_W%d", R, B, H, W);
    return buf;
}

// Reverse-step implementation: a forced shape (tile shapes select the tile
// kernel, strip shapes the strip kernel of that height; the reverse strip
// has one column per lane), else the tuned choice for this problem size, else the timing of one reverse step of each
// on the caller's data (t holds real buffers; what it writes is scratch).
static int adjoint_shape(const eed4_params *p, RevStep t, hipStream_t s, int *shape)
{
    TraceRange range("eed4 reverse-step shape %dx%dx%d", t.B, t.H, t.W);
    if (model_of_flags(p->flags) != 0) { *shape = kShapeStripShort; return EED4_OK; }
    const int forced = (p->flags >> 8) & 0xff;
    if (forced >= 1 && forced <= kNumShapes) { *shape = forced - 1; return EED4_OK; }
    if (p->flags & EED4_TILE_KERNEL) { *shape = 0; return EED4_OK; }
    const std::string key = adjoint_tune_key(t.R, t.B, t.H, t.W);
    if (tune_lookup(key, shape)) return EED4_OK;
    // the wide forward shapes map onto the same reverse strips as their heights
    const int cands[] = {kShapeStrip, kShapeStripTall, kShapeStripShort, kShapeStripTiny, 0, 1, 2};
    // The step is timed alone but runs beside the recompute, where instructions count:
    // short segments and tiles, which issue more of them, have to be clearly faster.
    // 2048^2 at R = 6: the tile 39 us alone against the 28-row strips' 38, the whole
    // backward 1830 us against 1700; 2700x2900 at R = 8, 80 rows 2110 us, 28 rows 2340.
    float margins[sizeof(cands) / sizeof(cands[0])];
    for (float &m : margins) m = kTuneMarginRefetch;
    const size_t N = (size_t)t.B * t.H * t.W;
    // every candidate reads the presmoothed state t.v
    const StepArgs a0 = make_args(p->sigma, t.R, p->tau, p->lambda, 0, model_of_flags(p->flags));
    hipError_t e = launch_blur(t.R, t.u, const_cast<float *>(t.v), t.B, t.H, t.W, a0, s);
    if (e == hipSuccess) e = launch_fill(t.ac, N, 0.0f, s);
    if (e != hipSuccess) return hip_fail(e, "adjoint autotune");
    int best = cands[0];
    const int rc = tune_pick(
        cands, (int)(sizeof(cands) / sizeof(cands[0])), s,
        [&](int c) {
            t.shape = c;
            t.first = 0;
            t.fresh = 0;                       // ac was cleared above
            return (int)EED4_OK;
        },
        [&](int, hipStream_t q) { return launch_reverse_step(t, p, p->cycle_len - 1, q); },
        "adjoint autotune", &best, nullptr, margins);
    if (rc != EED4_OK) return rc;
    tune_remember(key, best);
    *shape = best;
    return EED4_OK;
}

}  // namespace eed4

using namespace eed4;

extern "C" int eed4_backward(const float *ckpt, const uint8_t *mask, const float *known, int B,
                             int H, int W, const eed4_params *p, int M, const float *grad_u,
                             float *grad_known, float *grad_init, float *grad_lambda, void *ws,
                             size_t ws_bytes, void *stream)
{
    TraceRange range("eed4_backward %dx%dx%d, %d cycles of %d", B, H, W, M, p ? p->cycle_len : 0);
    int rc = check_params(p, B, H, W);
    if (rc != EED4_OK) return rc;
    if (!ckpt || !mask || !known || !grad_u || !grad_known || !grad_init || !grad_lambda || M < 1)
        return EED4_EINVAL;
    const int n = p->cycle_len, R = eed4_radius(p->sigma);
    BackwardLayout L = backward_layout(B, H, W, n, R);
    if ((rc = check_ws(ws, ws_bytes, L.total)) != EED4_OK) return rc;
    char *base = (char *)ws;
    hipStream_t s = (hipStream_t)stream;
    const size_t N = (size_t)B * H * W;
    float *Ubuf = (float *)(base + L.U);
    float *lp = (float *)(base + L.lp), *cyc = (float *)(base + L.cyc);
    float *slots = (float *)(base + L.slots);
    RevStep t{};
    t.an = (float *)(base + L.an);
    t.ac = (float *)(base + L.ac);
    t.ap = (float *)(base + L.ap);
    t.mask = mask;
    t.lp = lp;
    t.ls = n * max_adjoint_items(R, H, W);     // the tuner's steps below write within this
    t.B = B;
    t.H = H;
    t.W = W;
    t.R = R;
    const int fshape = run_shape(p, B, H, W);      // forward recompute
    hipError_t e;
#define EED4_TRY(x, what)                                    \
    do {                                                     \
        e = (x);                                             \
        if (e != hipSuccess) return hip_fail(e, what);       \
    } while (0)

    float *Vbuf = (float *)(base + L.V);
    {   // choose the reverse-step kernel (the timing runs write only scratch)
        RevStep probe = t;
        probe.u = ckpt + (size_t)(M - 1) * N;
        probe.an = grad_u;
        probe.v = Vbuf;
        if ((rc = adjoint_shape(p, probe, s, &t.shape)) != EED4_OK) return rc;
    }
    const int items = adjoint_items(R, t.shape, H, W);
    t.ls = n * items;
    EED4_TRY(hipMemcpyAsync((void *)t.an, grad_u, sizeof(float) * N, hipMemcpyDeviceToDevice, s),
             "seed copy");

    // The recompute of cycle m-1 (from its checkpoint) does not depend on the
    // reverse sweep of cycle m: it runs on a second stream into the other
    // buffer set.  rec[j] marks set j recomputed, done[j] marks the reverse
    // sweep that read set j finished (a stream wait takes the event's latest
    // record at the time of the call, so two of each suffice).
    hipStream_t s1 = recompute_stream();
    if (!s1) return hip_fail(hipErrorInvalidValue, "recompute stream");
    hipEvent_t ev[5] = {};
    for (auto &x : ev) {
        e = hipEventCreateWithFlags(&x, hipEventDisableTiming);
        if (e != hipSuccess) {
            for (auto &y : ev) if (y) (void)hipEventDestroy(y);
            return hip_fail(e, "event");
        }
    }
    hipEvent_t *rec = ev, *done = ev + 2, start = ev[4];
    const size_t nU = (size_t)(n > 1 ? n - 1 : 1);
    float *Uset[2] = {Ubuf, Ubuf + nU * N};
    float *Vset[2] = {Vbuf, Vbuf + (size_t)n * N};
    std::vector<const float *> Ur[2] = {std::vector<const float *>(n), std::vector<const float *>(n)};
    // u^{m,1..n-1} from the checkpoint, on s1, and v^{m,k} =
    // K_sigma * u^{m,k} for k = 0 .. n-1: the steps keep the v they compute, and
    // the last one, which no recomputed step forms, comes from the blur kernel
    auto recompute = [&](int m) -> hipError_t {
        trace_mark("eed4 recompute of cycle %d queued", m);
        std::vector<const float *> &U = Ur[m & 1];
        float *V = Vset[m & 1];
        U[0] = ckpt + (size_t)m * N;
        for (int k = 0; k + 1 < n; ++k) {
            float *out = Uset[m & 1] + (size_t)k * N;
            StepArgs a = make_args(p->sigma, R, p->tau, p->lambda, k, model_of_flags(p->flags));
            hipError_t r = launch_step_keepv(R, fshape, U[k], U[k > 0 ? k - 1 : 0], out,
                                             V + (size_t)k * N, mask, B, H, W, a, s1);
            if (r != hipSuccess) return r;
            U[k + 1] = out;
        }
        const StepArgs a = make_args(p->sigma, R, p->tau, p->lambda, 0, model_of_flags(p->flags));
        const hipError_t r = launch_blur(R, U[n - 1], V + (size_t)(n - 1) * N, B, H, W, a, s1);
        if (r != hipSuccess) return r;
        return hipEventRecord(rec[m & 1], s1);
    };
    float *an = (float *)t.an, *ac = t.ac, *ap = t.ap;
    int rc2 = EED4_OK;
#define EED4_TRY2(x, what)                                                  \
    if (rc2 == EED4_OK && (e = (x)) != hipSuccess) rc2 = hip_fail(e, what)
    EED4_TRY2(hipEventRecord(start, s), "event record");      // the seed and the checkpoints
    EED4_TRY2(hipStreamWaitEvent(s1, start, 0), "stream wait");
    EED4_TRY2(recompute(M - 1), "recompute step");
    for (int m = M - 1; m >= 0 && rc2 == EED4_OK; --m) {
        trace_mark("eed4 reverse sweep of cycle %d queued", m);
        EED4_TRY2(hipStreamWaitEvent(s, rec[m & 1], 0), "stream wait");
        if (m >= 1) {
            // set (m-1) & 1 was last read by the reverse sweep of cycle m+1
            if (m + 1 <= M - 1) EED4_TRY2(hipStreamWaitEvent(s1, done[(m + 1) & 1], 0), "stream wait");
            EED4_TRY2(recompute(m - 1), "recompute step");
        }
        const std::vector<const float *> &U = Ur[m & 1];
        for (int k = n - 1; k >= 0 && rc2 == EED4_OK; --k) {
            t.u = U[k];
            t.v = Vset[m & 1] + (size_t)k * N;
            t.an = an;
            t.ac = ac;
            t.ap = ap;
            t.first = k == 0 ? 1 : 0;
            t.fresh = k == n - 1 ? 1 : 0;          // ubar^{n-1} starts at 0
            t.lp = lp + (size_t)k * items;
            EED4_TRY2(launch_reverse_step(t, p, k, s), "reverse step");
            // ubar^k is complete in ac; ap holds the start of ubar^{k-1}
            float *tmp = an;
            an = ac;
            ac = ap;
            ap = tmp;
        }
        EED4_TRY2(hipEventRecord(done[m & 1], s), "event record");
        // this cycle's lambda partials: pairwise sum per image, then into the cascade
        const int j = M - 1 - m;                              // cycles summed before this one
        int carries = 0;
        while ((j >> carries) & 1) ++carries;
        const long long np = (long long)n * items;
        if (np <= 2048) {
            EED4_TRY2(launch_batches(B, 1, 1, 1024,
                                     [&](int b0, int, unsigned blocks) {
                                         hipLaunchKernelGGL(lambda_cycle_kernel, dim3(blocks),
                                                            dim3(1024), 0, s, lp, np, slots, b0, B,
                                                            carries);
                                     }),
                      "lambda sum");
        } else {
            EED4_TRY2(launch_pairwise_sum(lp, np, B, (float *)(base + L.t1),
                                          (float *)(base + L.t2), cyc, s), "lambda sum");
            EED4_TRY2(launch_lambda_carry(cyc, slots, B, carries, s), "lambda cascade");
        }
    }
#undef EED4_TRY2
    // on an error the recompute stream may still hold queued work on the
    // caller's workspace: let it finish before the caller can free it
    if (rc2 != EED4_OK) (void)hipStreamSynchronize(s1);
    for (auto &x : ev) (void)hipEventDestroy(x);
    if (rc2 != EED4_OK) return rc2;
    EED4_TRY(launch_adjoint_final(an, mask, grad_known, grad_init, N, s), "final");
    EED4_TRY(launch_lambda_final(slots, B, M, grad_lambda, s), "lambda final");
#undef EED4_TRY
    return EED4_OK;
}
