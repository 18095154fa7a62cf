// Internal: the plan object behind dmas_plan_t, and helpers shared by the
// host API (dmas_api.hip) and the serving runtime (dmas_server.hip).
#pragma once

#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <cmath>
#include <cstddef>
#include <cstdint>

#include "dmas.h"
#include "dmas_internal.hpp"

namespace dmas {
// Source of plan serial numbers, in creation order.
inline std::atomic<uint64_t> &plan_serials()
{
    static std::atomic<uint64_t> next{1};
    return next;
}
}  // namespace dmas

struct dmas_plan_s {
    uint64_t serial = dmas::plan_serials().fetch_add(1);   // creation order
    int device = 0;
    int cus = 0;           // its compute units
    int M = 0, T = 0, D = 0, order = 0;
    bool cf = true, nearfield = false, linear = false;
    bool roots = false;    // kernel reads a root plane (whole-sample delays, n >= 2)
    int pad0 = 0, pad1 = 0;   // zero pairs before and after a row of single calls' root planes
    // single calls that take the roots while staging, without a root plane: RF
    // images, envelopes, envelopes that allocate nothing
    bool direct_rf = false, direct_env = false, direct_noalloc = false;
    bool tables = false;   // per-tile delay tables (whole-sample delays, <= 2 GiB)
    bool block_tables = false;   // tables read a block of offsets at a time (kDelayTableBlocks)
    bool share_rings = false;    // with them, the envelope rings in the window region (...Shared)
    int compensated = 0;   // 0 FP32 sums, 1 Kahan FP32, 2 FP64
    int ng_fp64 = 0;
    int dtype = DMAS_F32;
    double fs = 0, c = 0;
    float cf_eps = 0;
    int fir_len = 0;
    int num_tiles = 0;
    int halo = 0;          // largest |delay - reference direction's| within a tile
    int range = 0;         // largest range of a microphone's delays within a tile
    int mic_block = 0;
    int direct_block = 0;  // microphones per LDS block of the launches without a root plane
    int row = 0;
    bool two_pass = false; // envelope calls: RF image into the output, then the filter over it in place
    int seg_rf = 0, seg_env = 0;   // samples per workgroup of a launch
    int nseg_rf = 0, nseg_env = 0;
    int seg_walk = 0, nseg_walk = 0;   // RF frames: those of a resident worker, and what a server counts
    size_t lds_rf = 0, lds_env = 0;
    int occ_rf = 0, occ_env = 0;
    double *d_mic = nullptr;
    double *d_dirs = nullptr;
    int32_t *d_tiles = nullptr;
    int32_t *d_tile_off = nullptr;    // per-tile delay tables (whole-sample delays), or null
    int32_t *d_tile_dref = nullptr;   // (in the allocation of d_tile_off)
    float *d_taps = nullptr;
    int env_decim = 1;
    int mf_len = 0;
    float *d_pulse = nullptr;
    size_t device_bytes = 0;   // all device memory the plan holds (geometry, taps, tiles, tables)
};

namespace dmas {

// Device bytes of a frame's root plane (zero when the plan does not use one).
inline size_t plane_bytes(const dmas_plan_s *plan)
{
    return plan->roots ? (size_t)plan->M * (size_t)plan->T * sizeof(float2) : 0;
}

// The same with the rows padded.
inline size_t padded_plane_bytes(const dmas_plan_s *plan)
{
    return plan->roots ? (size_t)plan->M * ((size_t)plan->pad0 + (size_t)plan->T + (size_t)plan->pad1) * sizeof(float2)
                       : 0;
}

// Zero pairs around the rows of single calls' root planes, so that windows
// reaching past the record's ends are copied like all others instead of
// element by element, which took several times as long: workgroups at the ends
// outlasted the rest (517 microphones, 361 x 4096 at order 2: 157 us against
// 100 us each, and the launch lasted as long as they did). A chunk starts at a
// sample of [0, T), its windows at most max_delay (samples, either way) and,
// without tables, the halo before it; the copy is `row` pairs long. Rows that
// would more than double (plus 1024 samples) stay unpadded, and so do planes
// that the padding would make kMaxPadBytes longer (short records of very many
// microphones: it would be most of their plane).
constexpr int64_t kMaxPadBytes = (int64_t)256 << 20;
inline void plane_pads(dmas_plan_s *plan, double max_delay)
{
    const double reach = std::ceil(max_delay * (1.0 + 1e-5)) + 2.0;
    const int halo = plan->tables ? 0 : plan->halo;
    const double before = reach + halo, after = std::max(0.0, reach - halo + plan->row);
    plan->pad0 = plan->pad1 = 0;
    if (before + after + 6 > (double)plan->T + 1024) return;
    const int pad0 = ((int)before + 3) & ~3, pad1 = ((int)after + 3) & ~3;
    if ((int64_t)plan->M * (pad0 + pad1) * (int64_t)sizeof(float2) > kMaxPadBytes) return;
    plan->pad0 = pad0;
    plan->pad1 = pad1;
}

// Memory for a call's root plane from alloc(void **, bytes): with the rows
// padded, or without where the device has no room for the padding.
template <class Alloc>
inline hipError_t allocate_plane(const dmas_plan_s *plan, Alloc &&alloc, float2 **plane, bool *padded)
{
    const size_t plain = plane_bytes(plan), full = padded_plane_bytes(plan);
    void *mem = nullptr;
    *padded = true;
    hipError_t e = alloc(&mem, full);
    if (e == hipErrorOutOfMemory && full > plain) {
        (void)hipGetLastError();
        *padded = false;
        e = alloc(&mem, plain);
    }
    *plane = e == hipSuccess ? static_cast<float2 *>(mem) : nullptr;
    return e;
}

// Output samples per workgroup of an RF launch: segments share nothing, so a cut
// costs only the workgroup's setup. (A server's grouping counts such frames as
// the long walks of plan_walks, which its caps are set for, and resident workers,
// which claim them one at a time, take those. 48 mixed RF frames of 16-64
// microphones 2.66 ms batched, counted as segments 2.93, both in walks 2.82; 7.9
// ms resident, in segments 10.3.) One to three chunks, so that each of
// `slots` places gets four workgroups where the record allows; more where the
// launch would not hold the workgroups (kMaxWorkgroups: with three chunks,
// images of 5e10 pixels and up). fixed > 0: that many, rounded up to 32.
inline void choose_rf_segments(int T, int num_tiles, int64_t slots, int fixed, int *seg, int *nseg)
{
    int s = (fixed + 31) & ~31;
    if (fixed <= 0) {
        const int64_t all = ((int64_t)T + kChunk - 1) / kChunk;
        int64_t chunks = 3;
        while (chunks > 1 && (int64_t)num_tiles * ((T + chunks * kChunk - 1) / (chunks * kChunk)) < 4 * slots) --chunks;
        const int64_t most = std::max<int64_t>(kMaxWorkgroups / num_tiles, 1);   // segments a tile
        s = (int)(std::max(chunks, (all + most - 1) / most) * kChunk);
    }
    *seg = s;
    *nseg = (T + s - 1) / s;
}

// Fill the root plane of input d_x (plans with roots only).
inline hipError_t stage_roots(const dmas_plan_s *plan, const void *d_x, float2 *d_plane, bool padded,
                              hipStream_t stream)
{
    return launch_roots(plan->order, plan->dtype, d_x, d_plane, plan->M, plan->T, padded ? plan->pad0 : 0,
                        padded ? plan->pad1 : 0, stream);
}

// Kernel arguments for one launch of `plan` on input d_x (and its root plane
// d_plane when the plan uses one) / output d_out.
inline KernelParams make_params(const dmas_plan_s *plan, const void *d_x, const float2 *d_plane, float *d_out,
                                float in_scale, bool env, bool padded = false)
{
    KernelParams kp{};
    kp.x = d_x;
    kp.roots = d_plane && padded ? d_plane + plan->pad0 : d_plane;
    kp.plane_lo = padded ? -plan->pad0 : 0;
    kp.plane_hi = plan->T + (padded ? plan->pad1 : 0);
    kp.plane_stride = kp.plane_hi - kp.plane_lo;
    kp.out = d_out;
    kp.mic = plan->d_mic;
    kp.dirs = plan->d_dirs;
    kp.tile_dirs = plan->d_tiles;
    kp.tile_off = plan->d_tile_off;
    kp.tile_dref = plan->d_tile_dref;
    kp.taps = plan->d_taps;
    kp.M = plan->M;
    kp.T = plan->T;
    kp.D = plan->D;
    kp.order = plan->order;
    kp.fir_len = env ? plan->fir_len : 1;
    kp.num_tiles = plan->num_tiles;
    kp.seg_len = env ? plan->seg_env : plan->seg_rf;
    kp.halo = plan->tables ? 0 : plan->halo;   // tables hold the window starts
    kp.row = plan->row;
    kp.mic_block = kp.table_block = plan->mic_block;
    kp.dtype = plan->dtype;
    kp.ng_fp64 = plan->ng_fp64;
    kp.fs = plan->fs;
    kp.c = plan->c;
    kp.cf_eps = plan->cf_eps;
    kp.in_scale = in_scale;
    kp.env_decim = env ? plan->env_decim : 1;
    kp.out_T = env ? (plan->T + plan->env_decim - 1) / plan->env_decim : plan->T;
    return kp;
}

inline LaunchShape shape_of(const dmas_plan_s *p, bool env)
{
    LaunchShape ls{};
    ls.order = p->order;
    ls.cf = p->cf;
    ls.env = env;
    ls.nearfield = p->nearfield;
    ls.delay = p->linear ? kDelayLinear
               : !p->tables ? kDelayComputed
               : !p->block_tables ? kDelayTable
               : p->share_rings   ? kDelayTableBlocksShared
                                  : kDelayTableBlocks;
    ls.accumulate = p->compensated;
    ls.grid = (unsigned)((int64_t)p->num_tiles * (env ? p->nseg_env : p->nseg_rf));
    ls.lds_bytes = env ? p->lds_env : p->lds_rf;
    return ls;
}

// The launch of a call without a root plane (no rings in the window region: that
// layout is for launches that fill the device).
inline LaunchShape direct_shape_of(const dmas_plan_s *p, bool env)
{
    LaunchShape ls = shape_of(p, env);
    ls.delay = kDelayTableDirect;
    ls.lds_bytes = (size_t)kernel_lds_bytes(p->direct_block, p->row, 2, env, (p->fir_len - 1) / 2, kDelayTableDirect);
    return ls;
}

// Its block, at most cap microphones, on tables built for blocks of mic_block:
// the whole array's rows lie one after another (mic_block >= M), or whole blocks
// make up one of the tables'.
inline int direct_block_of(int mic_block, int M, int cap)
{
    if (mic_block <= cap) return mic_block;
    if (mic_block >= M) return cap;
    int b = cap;
    while (mic_block % b) --b;
    return b;
}

// Workgroups of one launch of the plan.
inline int64_t plan_workgroups(const dmas_plan_s *p, bool env)
{
    return (int64_t)p->num_tiles * (env ? p->nseg_env : p->nseg_rf);
}

// The same with segments as long as the makespan allows: what a server counts a
// frame as, in device rounds, and the items of a resident worker.
inline int64_t plan_walks(const dmas_plan_s *p, bool env)
{
    return (int64_t)p->num_tiles * (env ? p->nseg_env : p->nseg_walk);
}

// Record the calling thread's last error message (returned by dmas_last_error).
void set_last_error(const char *msg);

// Launch one plan (order dispatch); with kp == nullptr, report occupancy in *blocks.
hipError_t launch_plan(int order, const KernelParams *kp, const LaunchShape &ls, hipStream_t st,
                       int *blocks = nullptr);

// Device time in us that taking the roots while staging adds to a call of the plan
// against reading a root plane (negative: it saves time), a fit to 220 frames of
// 4-128 microphones at orders 2-8 with 15-255 taps (residual 2.5 us; the time
// without a plane was 0.75 to 1.4 times that with one). Root pass and launch cost 2.4 us. A
// workgroup waits for its loads at every block of every chunk, 0.65 us longer than
// for copies from a plane; and a sample's root is taken again in every window that
// holds it, 1.1 us per 1e7 window elements, with Kahan and FP64 sums 1.85.
// occupancy: workgroups of the launch without a plane that a compute unit holds.
inline double direct_extra_us(const dmas_plan_s *p, bool env, int occupancy)
{
    const bool fused = env && !p->two_pass;
    const int seg = fused ? p->seg_env : p->seg_rf, nseg = fused ? p->nseg_env : p->nseg_rf;
    const int H = fused ? (p->fir_len - 1) / 2 : 0, lead = fused ? env_lead(H) : 0;
    if (nseg > 100000) return 1e9;
    int64_t chunks = 0, longest = 0;
    for (int s = 0; s < nseg; ++s) {
        const int64_t g0 = (int64_t)s * seg, g1 = std::min<int64_t>(g0 + seg, p->T);
        const int64_t n = (std::min<int64_t>(g1 + H, p->T) - std::max<int64_t>(g0 - lead, 0) + kChunk - 1) / kChunk;
        chunks += n;
        longest = std::max(longest, n);
    }
    const int64_t places = (int64_t)std::max(occupancy, 1) * std::max(p->cus, 1), workgroups = (int64_t)p->num_tiles * nseg;
    const int64_t blocks = (p->M + p->direct_block - 1) / p->direct_block;
    const double steps = (double)((workgroups + places - 1) / places) * (double)longest * (double)blocks;
    const double elements = (double)p->num_tiles * p->M * (double)chunks * p->row;
    return 0.65 * steps + (p->compensated ? 1.85e-7 : 1.1e-7) * elements - 2.4;
}

// Whether a call takes the roots while staging: the plan's choice, but not where
// the output shares memory with the channels, which a root plane copies first.
inline bool call_direct(const dmas_plan_s *p, const void *d_x, const float *d_out, bool env, bool noalloc)
{
    const size_t in = (size_t)p->M * (size_t)p->T * (p->dtype == DMAS_F32 ? 4 : 2);
    const size_t T = env ? ((size_t)p->T + p->env_decim - 1) / p->env_decim : (size_t)p->T;
    const uintptr_t x = reinterpret_cast<uintptr_t>(d_x), y = reinterpret_cast<uintptr_t>(d_out);
    const bool apart = x + in <= y || y + (size_t)p->D * T * sizeof(float) <= x;
    return apart && (!env ? p->direct_rf : noalloc ? p->direct_noalloc : p->direct_env);
}

// Launch the beamformer of one call and, for an envelope in two passes, the
// filter over its image (d_plane filled before, in stream order).
// direct: without a root plane.
inline hipError_t launch_image(const dmas_plan_s *plan, const void *d_x, const float2 *d_plane, bool padded,
                               bool direct, float *d_out, float in_scale, bool env, hipStream_t stream)
{
    const bool fused = env && !plan->two_pass;
    KernelParams kp = make_params(plan, d_x, d_plane, d_out, in_scale, fused, padded);
    const LaunchShape ls = direct ? direct_shape_of(plan, fused) : shape_of(plan, fused);
    if (direct) kp.mic_block = plan->direct_block;
    hipError_t e = launch_plan(plan->order, &kp, ls, stream);
    if (e == hipSuccess && env && !fused)
        e = launch_envelope_rows(d_out, plan->d_taps, plan->D, plan->T, plan->fir_len, plan->seg_env, plan->cus,
                                 stream);
    return e;
}

}  // namespace dmas
