// Host-side helpers shared by the translation units of libeed4.
#pragma once

#include "eed4.h"
#include "eed4_internal.h"

#include <rocprofiler-sdk-roctx/roctx.h>

#include <algorithm>
#include <cmath>
#include <cstdio>
#include <functional>
#include <string>

namespace eed4 {

// Host-side roctx ranges and marks around the library's calls, cycles and
// waits (`rocprofv3 --marker-trace` shows them beside the kernel trace).  A
// range lasts for the lifetime of the object.  Without a tool attached each
// costs a formatted string and a call that returns at once.
class TraceRange {
public:
    template <typename... A>
    explicit TraceRange(const char *fmt, A... a)
    {
        char buf[160];
        std::snprintf(buf, sizeof(buf), fmt, a...);
        roctxRangePushA(buf);
    }
    ~TraceRange() { roctxRangePop(); }
    TraceRange(const TraceRange &) = delete;
    TraceRange &operator=(const TraceRange &) = delete;
};

template <typename... A>
inline void trace_mark(const char *fmt, A... a)
{
    char buf[160];
    std::snprintf(buf, sizeof(buf), fmt, a...);
    roctxMarkA(buf);
}

// One FSI cycle over a batch of B equal-size images.
struct CycleJob {
    float *S, *X, *Y;          // S: cycle start; X, Y: rotation buffers
    float *Out = nullptr;      // where the last step writes u^{m,n}: S (in place) when null
    const uint8_t *mask;
    int B, H, W, R, shape, n;
    float sigma, tau, lambda;
    int model;                 // tensor variant (0: FOEED)
    double *partials;          // per-tile residual partials
    double *sums;              // [B][2] residual sums
    bool residual = true;      // form the cycle's residual sums
};

extern thread_local std::string g_last_hip;
int hip_fail(hipError_t e, const char *where);
size_t align_up(size_t x);
int check_params(const eed4_params *p, int B, int H, int W);
int check_ws(void *ws, size_t ws_bytes, size_t need);
int step_shape(const eed4_params *p, int B, int H, int W);
int run_shape(const eed4_params *p, int B, int H, int W);

// Without a tuned choice, the single-image path uses workgroup tiles when the
// problem has fewer 60 x 64 blocks than this, and strips otherwise.  Measured,
// 60 x 32 tiles against the strips: 2048^2 (1120 blocks) 17.6 against 21.5 us at
// R = 3, 23.0 against 28.4 at R = 8; 2560^2 (1720) 24.5 against 21.9 and 31.1
// against 30.4; 4096^2 55.5 against 43.6 and 68.8 against 55.2.
constexpr long long kMinStripBlocks = 1700;
// Images 29 to 32 wide need two 32 x 32 tiles across (28 output columns each), the
// second nearly empty, and one strip: from this many blocks on they run 8-row
// strips.  Tiles against strips, us a step at R = 2 / R = 8: 43 x 1024x29 (688
// blocks) 18.0 and 13.4 / 23.1 and 20.6, 84 x 1024x29 (1344) 28.8 and 20.4 / 37.5 and
// 29.3; 21 x 1024x29 (336) 9.8 and 8.3 / 12.9 and 12.1, but at R = 5 10.7 and 11.6.
constexpr long long kMinNarrowBlocks = 512;

// The autotuners keep the default shape unless another is faster by more than
// this factor, so shapes within timing noise of each other do not swap between
// runs.
constexpr float kTuneMargin = 0.98f;
// Candidate order for a tuner: `first`, then the other shapes in index order.
inline void tune_order(int first, int (&order)[kNumShapes])
{
    int n = 0;
    order[n++] = first;
    for (int sh = 0; sh < kNumShapes; ++sh)
        if (sh != first) order[n++] = sh;
}

// Candidates of the single-image tuner, `first` (the size rule's default)
// first; returns their count.  Where the default is a strip (enough work for
// the strips to fill the chip) only the 64 x 32 tile of the tiles is timed: it
// is level with the strips at about 7 million pixels (613x12000, R = 6: 30.5 us
// against 29.8) and 27 % slower at 4096^2.
// Where the default is a tile the 28- and 8-row strips are the strips that can
// compete.
inline int tune_candidates(int first, int (&order)[kNumShapes])
{
    int n = 0;
    order[n++] = first;
    for (int sh = 0; sh < kNumShapes; ++sh) {
        if (sh == first) continue;
        const bool keep = is_strip(first) ? is_strip(sh) || sh == 0
                                           : (!is_strip(sh) || sh == kShapeStripShort ||
                                              sh == kShapeStripTiny);
        if (keep) order[n++] = sh;
    }
    return n;
}
int default_step_shape(int R, int B, int H, int W);

// Margin a candidate of the single-image tuner must beat the current choice
// by.  Where the default is a strip (images large enough for it), the 28-row
// strips, which fetch more of the halo rows their neighbours share again, have
// to be clearly faster: in sustained runs they are at best level with the
// default (8 x 1037x771 at R = 3: 25.9 against 25.8 us; 2560^2 24.9 and 22.9),
// while a short tuning burst has at times put them a few percent ahead.  The tuner
// of the reverse step takes this margin for every shape but its default.
constexpr float kTuneMarginRefetch = 0.95f;
inline float tune_margin(int first, int shape)
{
    const bool refetch = shape == kShapeStripShort || shape == kShapeStripWideShort;
    return first == kShapeStrip && refetch ? kTuneMarginRefetch : kTuneMargin;
}

int capture_graph(const std::function<int(hipStream_t)> &enqueue, hipGraphExec_t *exec);

// Chooses one of n candidate shapes (cands[0] the default) by timing on stream
// s.  prepare(shape) sets up a candidate outside the timed region (EED4 code);
// launch(shape, stream) enqueues one launch of it.  A caller who solves a size
// once pays for all of this, so it takes few launches:
//  - A sample is some untimed work, which keeps the GPU busy while the host
//    queues the rest, and then the timed launches: about 100 us of them, at most
//    four, launched directly; or, where the default's launch takes less than
//    kTuneGraphUs, about 40 us of them replayed from a graph, as they will run
//    (launched one by one, kernels of less than about 5 us all take as long as the
//    host needs to launch them: 16 x 256^2 got a shape 20 % slower than the best).
//  - Every candidate gets one sample, those within 30 % of the fastest a second
//    and those within 6 % a third, in round-robin passes, and keeps its fastest,
//    so the clock ramp at the start does not favour the candidates timed later.
// A candidate replaces the current choice only when it is faster by more than
// kTuneMargin (or its own entry of margins).
constexpr float kTuneGraphUs = 12.0f;
template <typename Prepare, typename Launch>
int tune_pick(const int *cands, int n, hipStream_t s, Prepare &&prepare, Launch &&launch,
              const char *where, int *best, float *best_ms, const float *margins = nullptr)
{
    hipEvent_t e0 = nullptr, e1 = nullptr;
    hipGraphExec_t exec[kNumShapes] = {};
    hipError_t e = hipEventCreate(&e0);
    if (e == hipSuccess) e = hipEventCreate(&e1);
    float tmin[kNumShapes];
    for (int i = 0; i < n; ++i) tmin[i] = 1e30f;
    int rc = EED4_OK;
    // ms of `count` launches of candidate i (of its graph where it has one)
    auto sample = [&](int i, int count) -> float {
        auto enqueue = [&](int c) {
            if (exec[i]) return hipGraphLaunch(exec[i], s);
            hipError_t le = hipSuccess;
            for (int l = 0; l < c && le == hipSuccess; ++l) le = launch(cands[i], s);
            return le;
        };
        float ms = 0.0f;
        e = enqueue(1);
        if (e == hipSuccess) e = hipEventRecord(e0, s);
        if (e == hipSuccess) e = enqueue(count);
        if (e == hipSuccess) e = hipEventRecord(e1, s);
        if (e == hipSuccess) e = hipEventSynchronize(e1);
        if (e == hipSuccess) e = hipEventElapsedTime(&ms, e0, e1);
        return ms;
    };
    float us = 0.0f;                                     // a launch of the default
    if (e == hipSuccess && (rc = prepare(cands[0])) == EED4_OK) us = std::fmax(500.0f * sample(0, 2), 1.0f);
    const bool graph = us < kTuneGraphUs;
    const int count = graph ? (int)std::fmin(8.0f, std::ceil(40.0f / us))
                            : (int)std::fmin(4.0f, std::ceil(100.0f / us));
    for (int pass = 0; pass < 3 && e == hipSuccess && rc == EED4_OK; ++pass) {
        constexpr float kWithin[3] = {1e30f, 1.3f, 1.06f};
        const float limit = kWithin[pass] * *std::min_element(tmin, tmin + n);
        for (int i = 0; i < n && e == hipSuccess && rc == EED4_OK; ++i) {
            if (pass > 0 && i > 0 && tmin[i] > limit) continue;      // the default stays in
            if ((rc = prepare(cands[i])) != EED4_OK) break;
            if (graph && !exec[i]) {
                rc = capture_graph(
                    [&](hipStream_t cs) {
                        for (int l = 0; l < count; ++l) {
                            const hipError_t le = launch(cands[i], cs);
                            if (le != hipSuccess) return hip_fail(le, where);
                        }
                        return (int)EED4_OK;
                    },
                    &exec[i]);
                if (rc != EED4_OK) break;
            }
            const float ms = sample(i, count);
            if (e == hipSuccess) tmin[i] = std::fmin(tmin[i], ms);
        }
    }
    if (rc != EED4_OK || e != hipSuccess) (void)hipStreamSynchronize(s);
    for (int i = 0; i < n; ++i)
        if (exec[i]) (void)hipGraphExecDestroy(exec[i]);
    if (e0) (void)hipEventDestroy(e0);
    if (e1) (void)hipEventDestroy(e1);
    if (rc != EED4_OK) return rc;
    if (e != hipSuccess) return hip_fail(e, where);
    int b = 0;
    for (int i = 1; i < n; ++i)
        if (tmin[i] < (margins ? margins[i] : kTuneMargin) * tmin[b]) b = i;
    *best = cands[b];
    if (best_ms) *best_ms = tmin[b] / count;
    return EED4_OK;
}

// Autotuner choice cache (process-wide; persisted to the file named by
// EED4_AUTOTUNE_CACHE when set).
bool tune_lookup(const std::string &key, int *shape);
void tune_remember(const std::string &key, int shape);
std::string single_tune_key(int R, int B, int H, int W);
int tune_single_step(const eed4_params *p, int B, int H, int W, float *S, float *X,
                     const uint8_t *mask, hipStream_t s, int *shape);
StepArgs make_args(float sigma, int R, float tau, float lambda, int k, int model = 0);
hipStream_t capture_stream();
hipStream_t recompute_stream();
void cycle_roles(int k, int n, float *S, float *X, float *Y, float **cur, float **prev,
                 float **out);
int enqueue_cycle(const CycleJob &j, hipStream_t s);
int capture_cycle(const CycleJob &j, hipGraphExec_t *exec, int nc = 1);
size_t backward_workspace(int B, int H, int W, const eed4_params *p);

}  // namespace eed4
