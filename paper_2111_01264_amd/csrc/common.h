// Shared host-side helpers of the DQN hot-path library: error reporting and launch checks.
#pragma once
#include <hip/hip_runtime.h>
#include <stdarg.h>
#include <stdint.h>
#include <stdio.h>

#include "../../include/dqn_mi355.h"
#include "philox.h"

namespace dqn {

// Thread-local message behind dqn_last_error().
char* error_buffer();
int fail(int code, const char* fmt, ...);

#define DQN_HIP(expr)                                                                        \
    do {                                                                                     \
        hipError_t e__ = (expr);                                                             \
        if (e__ != hipSuccess)                                                               \
            return ::dqn::fail(e__ == hipErrorOutOfMemory ? DQN_ENOMEM : DQN_EHIP,           \
                               "%s failed: %s", #expr, hipGetErrorString(e__));              \
    } while (0)

#define DQN_LAUNCH_CHECK()                                                                   \
    do {                                                                                     \
        hipError_t e__ = hipGetLastError();                                                  \
        if (e__ != hipSuccess)                                                               \
            return ::dqn::fail(DQN_EHIP, "kernel launch failed at %s:%d: %s", __FILE__,      \
                               __LINE__, hipGetErrorString(e__));                            \
    } while (0)

inline bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

// Replay internals needed by dqn_sync_target.
int replay_flush_ordered(replay* rb);
hipStream_t replay_sample_stream(replay* rb);
hipStream_t replay_push_stream(replay* rb);
int replay_lanes(const replay* rb);
// Context internals needed by the Algorithm 1 orchestrator.
hipStream_t dqn_ctx_act_stream(dqn_ctx* c);
int dqn_ctx_num_actions(const dqn_ctx* c);
int dqn_ctx_max_envs(const dqn_ctx* c);
int dqn_ctx_max_batch(const dqn_ctx* c);

constexpr int kFrameBytes = 84 * 84;          // 7056 = 441 * 16
constexpr int kFrameVec16 = kFrameBytes / 16; // 441
constexpr int kStateBytes = 4 * kFrameBytes;
constexpr int kMaxLanes = 64;

// A frame is 7056 = 110.25 x 64 bytes, so frames in a [n][84][84] array start at every 16-byte phase of a
// 64-byte line.  A 16-byte store whose group of four lanes straddles a line boundary reaches memory as two
// partial writes (measured: 1.75x the written bytes on average); shifting the vector index by the
// destination's phase makes every group of four lanes cover exactly one line.
__device__ inline int line_phase(const void* p) { return static_cast<int>((reinterpret_cast<uintptr_t>(p) >> 4) & 3); }

__device__ inline void copy_frame(uint8_t* __restrict__ dst, const uint8_t* __restrict__ src)
{
    const uint4* s = reinterpret_cast<const uint4*>(src);
    uint4* d = reinterpret_cast<uint4*>(dst);
    const int ph = line_phase(dst);
    for (int v = static_cast<int>(threadIdx.x) - ph; v < kFrameVec16; v += blockDim.x)
        if (v >= 0) d[v] = s[v];
}

// One experience per lane appended to the temporary buffers (Section 3), as data for a kernel: what
// replay_push_step does, for a caller that folds the append into a launch of its own.
struct PushStepPlan {
    const uint8_t* frames;      // [L][84][84]
    const int32_t* actions;     // [L]
    const float* rewards;       // [L]
    const uint8_t* terminals;   // [L]
    uint8_t* st_frames;
    int32_t* st_actions;
    float* st_rewards;
    uint8_t* st_terminals;
    int64_t S;                  // staging slots per lane
    int32_t L;                  // 0 = nothing to append
    int32_t slot[kMaxLanes];    // staging slot of each lane's new experience
};

// Workgroup `lane` of a push: frame copy by the whole workgroup, the three scalars by thread 0.
__device__ inline void push_step_block(const PushStepPlan& p, int lane)
{
    const int64_t dst = static_cast<int64_t>(lane) * p.S + p.slot[lane];
    copy_frame(p.st_frames + dst * kFrameBytes, p.frames + static_cast<int64_t>(lane) * kFrameBytes);
    if (threadIdx.x == 0) {
        p.st_actions[dst] = p.actions[lane];
        p.st_rewards[dst] = p.rewards[lane];
        p.st_terminals[dst] = p.terminals[lane];
    }
}

// The lanes as a gather sees them.  A lane of `count` visible frames holds count - 4 complete transitions (none if that is negative);
// entries past the last lane read end = V, so that a walk over whole groups of eight needs no other bound.
struct LaneTable {
    int32_t head[kMaxLanes];   // next write position inside the lane
    int32_t end[kMaxLanes];    // complete transitions in this lane and all before it (2^31 frames would be 15 TB)
};
static_assert(kMaxLanes % 8 == 0, "whole trips over the lanes' table");

// One replay_sample_gather call as data for a kernel (for a caller that folds the gather into a launch of its own).
struct GatherPlan {
    const uint8_t* frames; const int32_t* actions; const float* rewards; const uint8_t* terminals;   // the ring
    LaneTable tab;
    int32_t L; int64_t M, V;
    uint64_t seed, sample_step;
    const int64_t* idx_in;
    uint8_t* s; uint8_t* s2; int32_t* a; float* r; float* done; int64_t* idx_out;
    int32_t B;                  // 0 = nothing to gather
};

// The transition that draw b of the call selects (or that idx_in names): its global index, lane and age j in the lane, and
// whether its five-frame window (ages j-3 .. j+1) lies in the lane.  The chain in front of the frame's request is what a gather waits for, and
// a read of the kernel arguments is a round trip of its own: everything is read here at once (the empty asm statements keep the
// compiler from moving the reads to where they are used), the walk over the lanes is selects on eight entries at a time, and there is
// no 64-bit division (ring positions wrap by one subtraction, see window_slot).
struct SampledRow {
    int64_t idx, j;
    int64_t lane0, base, M;   // first slot of the lane; ring position of its oldest frame, in [0, 2 M); slots per lane
    bool ok;
};
__device__ inline SampledRow sampled_row(const GatherPlan& p, int b)
{
    SampledRow r;
    const uint64_t seed = p.seed, step = p.sample_step;
    const int64_t V = p.V, M = p.M;
    const int32_t L = p.L;
    const int64_t* idx_in = p.idx_in;
    int32_t e8[8], h8[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) { e8[q] = p.tab.end[q]; h8[q] = p.tab.head[q]; }
    asm volatile("" :: "s"(seed), "s"(step), "s"(V), "s"(M), "s"(L), "s"(idx_in));
    asm volatile("" :: "s"(e8[0]), "s"(e8[1]), "s"(e8[2]), "s"(e8[3]), "s"(e8[4]), "s"(e8[5]), "s"(e8[6]), "s"(e8[7]));
    asm volatile("" :: "s"(h8[0]), "s"(h8[1]), "s"(h8[2]), "s"(h8[3]), "s"(h8[4]), "s"(h8[5]), "s"(h8[6]), "s"(h8[7]));
    int32_t start = 0, end = 0, head = 0, lane = 0;
    if (idx_in) {
        r.idx = idx_in[b];
        r.ok = r.idx >= 0 && r.idx < static_cast<int64_t>(L) * M;
        lane = r.ok ? static_cast<int>(r.idx / M) : 0;
        r.j = r.ok ? r.idx - lane * M : 0;
        start = lane > 0 ? p.tab.end[lane - 1] : 0;
        end = p.tab.end[lane];
        head = p.tab.head[lane];
    } else {
        const Philox4 d = philox_draw(seed, kTagSample, step, static_cast<uint32_t>(b));
        const uint64_t u = (static_cast<uint64_t>(d.x[1]) << 32) | d.x[0];
        int32_t k = static_cast<int32_t>(__umul64hi(u, static_cast<uint64_t>(V)));
        asm("" : "+v"(k));   // vector selects also where the draw is the same for a whole workgroup: scalar ones become branches
        auto walk = [&](int l0, const int32_t (&e)[8], const int32_t (&hd)[8]) {
#pragma unroll
            for (int q = 0; q < 8; ++q) {   // lane l0 + q, if the draw lies past every lane before it
                const bool past = k >= end;
                start = past ? end : start;
                head = past ? hd[q] : head;
                lane = past ? l0 + q : lane;
                end = past ? e[q] : end;
            }
        };
        walk(0, e8, h8);    // (end = 0 before the first lane)
        for (int l0 = 8; l0 < L; l0 += 8) {
            int32_t e[8], hd[8];
#pragma unroll
            for (int q = 0; q < 8; ++q) { e[q] = p.tab.end[l0 + q]; hd[q] = p.tab.head[l0 + q]; }
            walk(l0, e, hd);
        }
        r.j = 3 + (k - start);
        r.idx = lane * M + r.j;
        r.ok = true;
    }
    const int32_t count = end - start + 4;   // (a lane with fewer than five frames holds no valid age)
    r.ok = r.ok && r.j >= 3 && r.j <= static_cast<int64_t>(count) - 2;
    r.lane0 = lane * M;
    r.M = M;
    r.base = static_cast<int64_t>(head) - count + M;
    return r;
}
// Slot of the frame of age j - 3 + u of a valid row, 0 <= u <= 4: head + M - 1 is the newest frame's position before the wrap, so one
// subtraction wraps.
__device__ inline int64_t window_slot(const SampledRow& r, int u)
{
    const int64_t at = r.base + r.j - 3 + u;
    return r.lane0 + (at >= r.M ? at - r.M : at);
}
// The minibatch row of sample b as a DESCRIPTOR instead of copied frames: desc[0..3] = replay slots of the four frames
// of s, desc[4..7] = those of s', -1 for a frame that is all zeros (a terminal flag lies between it and the stack's
// newest frame, or the index is invalid); a, r, done (and idx_out) are written as gather_block writes them.  A kernel
// that consumes states can then read the frames straight from the replay memory (Section 2.1: states are stacks of
// the four latest frames), and the 56 KB per sample that a materialised (s, s') pair costs are never written.
constexpr int kDescInts = 8;
__device__ inline void sample_desc(const GatherPlan& p, int b, int32_t* __restrict__ desc)
{
    const SampledRow row = sampled_row(p, b);
    if (p.idx_out) p.idx_out[b] = row.idx;
    if (!row.ok) {
#pragma unroll
        for (int f = 0; f < kDescInts; ++f) desc[f] = -1;
        p.a[b] = -1; p.r[b] = 0.f; p.done[b] = 0.f;
        return;
    }
    int32_t slot[5];
#pragma unroll
    for (int f = 0; f < 5; ++f) slot[f] = static_cast<int32_t>(window_slot(row, f));
    const int32_t act = p.actions[slot[3]];
    const float rew = p.rewards[slot[3]];
    uint32_t t[4];   // terminal flags of ages j-3 .. j
#pragma unroll
    for (int u = 0; u < 4; ++u) t[u] = p.terminals[slot[u]];
#pragma unroll
    for (int f = 0; f < 4; ++f) {
        uint32_t any_s = 0, any_s2 = 0;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            if (u >= f && u <= 2) any_s |= t[u];          // frame f of s: ages j-3+f .. j-1
            if (u >= f + 1) any_s2 |= t[u];               // frame f of s' is window frame f+1: ages j-2+f .. j
        }
        desc[f] = any_s ? -1 : slot[f];
        desc[4 + f] = any_s2 ? -1 : slot[f + 1];
    }
    p.a[b] = act;
    p.r[b] = rew;
    p.done[b] = t[3] ? 1.f : 0.f;
}

// Workgroup (frame f of the five-frame window ages j-3 .. j+1, sample b), 256 threads.  The frame is written into s (position f,
// f <= 3) and s2 (position f-1, f >= 1), each zeroed if a terminal flag lies between the frame and the newest frame of that
// stack (Section 2.1: states are stacks of the four latest frames).  The chain is draw -> frame -> stores: the frame is
// requested together with the flags that decide whether it counts, everything of it at once.
__device__ inline void gather_block(const GatherPlan& p, int f, int b)
{
    uint8_t* s = p.s; uint8_t* s2 = p.s2;
    const uint8_t* frames = p.frames; const uint8_t* terminals = p.terminals;
    asm volatile("" :: "s"(s), "s"(s2), "s"(frames), "s"(terminals));
    SampledRow row = sampled_row(p, b);
    row.ok = __builtin_amdgcn_readfirstlane(row.ok);
    uint4* ds = reinterpret_cast<uint4*>(s + (static_cast<int64_t>(b) * 4 + (f <= 3 ? f : 0)) * kFrameBytes);
    uint4* ds2 = reinterpret_cast<uint4*>(s2 + (static_cast<int64_t>(b) * 4 + (f >= 1 ? f - 1 : 0)) * kFrameBytes);
    // each destination with its own phase shift (see copy_frame): the second read of the frame comes from cache
    const int v1 = static_cast<int>(threadIdx.x) - line_phase(ds), v2 = static_cast<int>(threadIdx.x) - line_phase(ds2);
    static_assert(kFrameVec16 + 3 <= 512, "two vectors per thread and destination");
    uint4 w1[2], w2[2];
    uint32_t keep_s = 0, keep_s2 = 0;
    if (row.ok) {   // uniform
        uint32_t t[4];   // terminal flags of ages j-3 .. j
#pragma unroll
        for (int u = 0; u < 4; ++u) t[u] = terminals[window_slot(row, u)];
        const uint4* src = reinterpret_cast<const uint4*>(frames + window_slot(row, f) * kFrameBytes);
        auto clamped = [](int v) { return v < 0 ? 0 : (v < kFrameVec16 ? v : kFrameVec16 - 1); };
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            w1[u] = src[clamped(v1 + 256 * u)];
            w2[u] = src[clamped(v2 + 256 * u)];
        }
        if (f == 0 && threadIdx.x == 0) {
            const int64_t tslot = window_slot(row, 3);
            p.a[b] = p.actions[tslot];
            p.r[b] = p.rewards[tslot];
            p.done[b] = t[3] ? 1.f : 0.f;
        }
        // a frame behind a terminal flag is zeroed with a mask (a choice between the loaded vector and a zero vector made the
        // compiler keep the zero vector in scratch memory and load through a pointer)
        uint32_t any_s = 0, any_s2 = 0;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            if (u >= f && u <= 2) any_s |= t[u];
            if (u >= f) any_s2 |= t[u];
        }
        keep_s = any_s ? 0u : 0xFFFFFFFFu;
        keep_s2 = any_s2 ? 0u : 0xFFFFFFFFu;
    } else {
#pragma unroll
        for (int u = 0; u < 2; ++u) w1[u] = w2[u] = make_uint4(0, 0, 0, 0);
        if (f == 0 && threadIdx.x == 0) { p.a[b] = -1; p.r[b] = 0.f; p.done[b] = 0.f; }
    }
#pragma unroll
    for (int u = 0; u < 2; ++u) {
        const int a1 = v1 + 256 * u, a2 = v2 + 256 * u;
        if (f <= 3 && a1 >= 0 && a1 < kFrameVec16) ds[a1] = make_uint4(w1[u].x & keep_s, w1[u].y & keep_s, w1[u].z & keep_s, w1[u].w & keep_s);
        if (f >= 1 && a2 >= 0 && a2 < kFrameVec16) ds2[a2] = make_uint4(w2[u].x & keep_s2, w2[u].y & keep_s2, w2[u].z & keep_s2, w2[u].w & keep_s2);
    }
    if (p.idx_out && f == 0 && threadIdx.x == 0) p.idx_out[b] = row.idx;
}

// Validates a replay_sample_gather call and fills `plan` without enqueuing anything.
int replay_plan_sample_gather(replay* rb, int32_t B, uint64_t sample_step, const int64_t* idx_in, uint8_t* s, uint8_t* s2,
                              int32_t* a, float* r, float* done, int64_t* idx_out, GatherPlan* plan);
// Changes with every flush (and differs between replay memories): two gathers of the same sample step read the same
// minibatch iff their epochs are equal.
uint64_t replay_epoch(const replay* rb);
// The ring's frame array [capacity][84][84] (device memory owned by rb).
const uint8_t* replay_ring_frames(const replay* rb);

// Validates a replay_push_step call and fills `plan` without enqueuing anything; replay_commit_push_step then
// records that the experiences have been appended (call it once the kernel carrying the plan is enqueued).
int replay_plan_push_step(replay* rb, const uint8_t* frames, const int32_t* actions, const float* rewards,
                          const uint8_t* terminals, PushStepPlan* plan);
void replay_commit_push_step(replay* rb);

}  // namespace dqn
