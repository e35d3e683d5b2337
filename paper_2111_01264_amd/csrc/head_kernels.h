// The non-GEMM kernels of the act and train steps: fc2 + epsilon-greedy, fc2 + TD target / loss
// (Eq. 1), fc2 backward, bias gradients, centered RMSProp (Appendix B) with the refresh of the
// operand copies, and the target copy (theta^- <- theta).
#pragma once
#include "common.h"
#include "conv_tower.h"
#include "vec4.h"
#include "philox.h"

namespace dqn {

constexpr int kMaxBatch = 1024;
constexpr int kMaxActions = 32;

// Offsets of the tensors inside a parameter blob (identical for the public and the device layout).
struct Offsets {
    size_t w1, b1, w2, b2, w3, b3, wf1, bf1, wf2, bf2, total;
};
// (all but the end of the blob are the same for every number of actions)
constexpr size_t kOffW1 = 0, kOffB1 = kOffW1 + 32 * 256, kOffW2 = kOffB1 + 32, kOffB2 = kOffW2 + 64 * 512, kOffW3 = kOffB2 + 64, kOffB3 = kOffW3 + 64 * 576,
                 kOffWf1 = kOffB3 + 64, kOffBf1 = kOffWf1 + 512 * 3136, kOffWf2 = kOffBf1 + 512;
inline Offsets make_offsets(int A)
{
    Offsets o;
    o.w1 = kOffW1;   o.b1 = kOffB1;   o.w2 = kOffW2;   o.b2 = kOffB2;   o.w3 = kOffW3;   o.b3 = kOffB3;
    o.wf1 = kOffWf1; o.bf1 = kOffBf1; o.wf2 = kOffWf2;
    o.bf2 = o.wf2 + static_cast<size_t>(A) * 512;
    o.total = o.bf2 + A;
    return o;
}

// Backward operand copies ("transposed shadows"), one buffer of T:
//   conv2: [4 parity classes][32 c][(p2, q2, o) = 256]   conv3: [64 c][(p, q, o) = 576]
//   fc1:   [3136 f][512 o]
// All three are kept in MFMA fragment order (over [row][k]: conv per (class,) [c][k], fc1 over [f][o]), the order their
// consumers load them in: one operand of a matrix instruction is then one contiguous 1 KB row instead of 16 or 32 separate
// cache lines.
// Full precision: conv2's and conv3's are behind the end, as three bf16 parts each (third_index) and with the taps reversed, see
// conv_tower_bwd_f32.h.
constexpr size_t kBshW2 = 0, kBshW3 = 4 * 32 * 256, kBshWf1 = kBshW3 + 64 * 576;
constexpr size_t kBshTotal = kBshWf1 + static_cast<size_t>(3136) * 512;

constexpr size_t kThirdsW2 = 0, kThirdsW3 = static_cast<size_t>(3) * 64 * 512, kThirdsTotal = kThirdsW3 + static_cast<size_t>(3) * 64 * 576;   // bf16 elements
inline size_t bsh_elements(size_t esize) { return kBshTotal + (esize == 4 ? kThirdsTotal / 2 : 0); }

// The value v as row o, column k of a [..][K] matrix in three bf16 parts whose sum it is: 8 + 8 + 8 significand bits.
__device__ inline void store_thirds(bf16_t* thirds, int o, int k, int K, float v)
{
#pragma unroll
    for (int q = 0; q < 3; ++q) {
        const bf16_t p = static_cast<bf16_t>(v);
        thirds[third_index(o, k, K, q)] = p;
        v -= static_cast<float>(p);
    }
}

// Element r of conv2.w ([o][p][q][c]) / conv3.w into the backward copy.
template <typename T> __device__ inline void bsh_store_w2(T* bsh, int r, float v)
{
    const int c = r % 32, q = (r / 32) % 4, p = (r / 128) % 4, oc = r / 512;
    const int cls = (p % 2) * 2 + (q % 2), tap = (p / 2) * 2 + (q / 2);
    if (sizeof(T) == 2) bsh[kBshW2 + static_cast<size_t>(cls) * 32 * 256 + tower_frag_index(c, tap * 64 + oc, 256)] = from_float<T>(v);
    else store_thirds(reinterpret_cast<bf16_t*>(bsh + kBshTotal) + kThirdsW2 + static_cast<size_t>(cls) * 3 * 32 * 256, c, (3 - tap) * 64 + oc, 256, v);
}
template <typename T> __device__ inline void bsh_store_w3(T* bsh, int r, float v)
{
    const int c = r % 64, q = (r / 64) % 3, p = (r / 192) % 3, oc = r / 576;
    const int tap = p * 3 + q;
    if (sizeof(T) == 2) bsh[kBshW3 + tower_frag_index(c, tap * 64 + oc, 576)] = from_float<T>(v);
    else store_thirds(reinterpret_cast<bf16_t*>(bsh + kBshTotal) + kThirdsW3, c, (8 - tap) * 64 + oc, 576, v);
}

template <typename T> __host__ __device__ inline size_t bsh_index_wf1(int o, int f)
{
    return kBshWf1 + frag_index<T>(f, o, 512);
}

// Full precision: conv2's and conv3's weights are not in the forward copy's own places but behind its end, as three bf16 parts each
// (third_index) whose sum is the fp32 weight: 8 + 8 + 8 significand bits.
__host__ __device__ inline size_t thirds_offset(const Offsets& off) { return (off.total + 63) / 64 * 64; }   // in floats
inline size_t copy_elements(const Offsets& off, size_t esize) { return esize == 4 ? thirds_offset(off) + kThirdsTotal / 2 : off.total; }

// Where blob element e lives in the forward copy: identical, except that the weights of fc1 and, in bf16 mode, of the conv layers are kept
// in MFMA fragment order of the kernels that load them (full precision: conv2's and conv3's are elsewhere, see shadow_store).  bf16
// mode stores conv1's weights as fp16 (that kernel runs conv1 on the f16 matrix instruction), everything else as bf16: shadow_store converts.
template <typename T> __host__ __device__ inline size_t shadow_index(const Offsets& off, size_t e)
{
    if (sizeof(T) == 2) {
        if (e >= off.w1 && e < off.b1) { const int r = static_cast<int>(e - off.w1); return off.w1 + tower_frag_index(r / 256, r % 256, 256); }
        if (e >= off.w2 && e < off.b2) { const int r = static_cast<int>(e - off.w2); return off.w2 + tower_frag_index(r / 512, r % 512, 512); }
        if (e >= off.w3 && e < off.b3) { const int r = static_cast<int>(e - off.w3); return off.w3 + tower_frag_index(r / 576, r % 576, 576); }
    }
    if (e >= off.wf1 && e < off.bf1) { const int r = static_cast<int>(e - off.wf1); return off.wf1 + frag_index<T>(r / 3136, r % 3136, 3136); }
    return e;
}

template <typename T> __device__ inline void shadow_store(T* sh, const Offsets& off, size_t e, float v)
{
    if (sizeof(T) == 2 && e >= off.w1 && e < off.b1) reinterpret_cast<_Float16*>(sh)[shadow_index<T>(off, e)] = static_cast<_Float16>(v);
    else if (sizeof(T) == 4 && ((e >= off.w2 && e < off.b2) || (e >= off.w3 && e < off.b3))) {
        const bool second = e < off.b2;
        const int r = static_cast<int>(e - (second ? off.w2 : off.w3)), K = second ? 512 : 576;
        store_thirds(reinterpret_cast<bf16_t*>(sh + thirds_offset(off)) + (second ? kThirdsW2 : kThirdsW3), r / K, r % K, K, v);
    }
    else sh[shadow_index<T>(off, e)] = from_float<T>(v);
}

// ---- network head, forward: finish fc1, fc2 on the matrix cores, then action selection (act step)
// or TD target / error / loss (train step, Eq. 1) -------------------------------------------------
//
// fc1 arrives as kFc1Slices k-slices of fp32 partial sums [groups][slice][rows][512].  A workgroup owns
// kHeadRows samples (few rows per workgroup: the slice sums are plain loads, and what bounds them is
// how many compute units pull at once).  (1) Thread t finishes four features of one row for every
// group -- slices added in slice order, bias, ReLU, rounded to the operand type so that forward and
// backward see the same h -- into an LDS tile; the fc2 weight fragments are requested before that,
// so both latencies overlap.  (2) Per group the four wavefronts each take a quarter of K = 512 of
// the fc2 product as 16x16 MFMAs (A = W2 rows, B = the h tile); the partial accumulators meet in LDS
// and are added in wavefront order.  (3) One wavefront runs the tail, 32 lanes per sample.
constexpr int kHeadRows = 2;
constexpr int kFc1Slices = 7;

struct HeadArgs {
    const float* partial;        // [groups][kFc1Slices][rows][512]
    int rows, A;
    int head_blocks;             // workgroups of the head proper (the first ones of the grid)
    const float* b1[3];
    const void* w2[3];           // T [A][512]
    const float* b2[3];
    // act step
    float epsilon;
    uint64_t seed, act_step;
    int32_t* actions;
    float* q_out;                // [rows][A] or null
    // train step
    const int32_t* act;
    const float* rew;
    const float* done;
    float gamma, huber;
    void* h_online;              // T [rows][512]: h of group 0, kept for the backward pass
    void* dzh;                   // T [rows][512]: dLoss/d(fc1 pre-activation) = dq_b W2[a_b][.] [h > 0]
    float* q_all;                // [groups][rows][A]
    float* dqv;
    float* lossv;
    // Train step: workgroups [head_blocks, head_blocks + 5 * gather.B) gather the NEXT minibatch from the replay memory
    // (D is constant between synchronisation points, Section 3): independent byte copies that would otherwise cost a
    // dependent launch of their own in front of every train step.  With desc_out set, the minibatch is only DESCRIBED
    // (sample_desc: replay slots per frame, a, r, done), by ceil(gather.B / 256) workgroups instead: the kernel that
    // consumes the states then reads the frames from the replay memory itself.  (Last in the struct: the act step
    // never reads it.)
    int32_t* desc_out;           // [gather.B][kDescInts] or null
    GatherPlan gather;
};

// fc2's operands for the 16x16 matrix instructions: a step is 16 rows x KS contraction elements, each lane holding E consecutive ones.
template <typename T> struct HeadMma;
template <> struct HeadMma<bf16_t> {
    typedef bf16x8 vec;
    static constexpr int KS = 32, E = 8;
    __device__ static void mma(f32x4v& acc, const vec& w, const vec& h) { acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w, h, acc, 0, 0, 0); }
};
template <> struct HeadMma<float> {
    typedef f32x4v vec;
    static constexpr int KS = 16, E = 4;
    __device__ static void mma(f32x4v& acc, const vec& w, const vec& h)
    {
#pragma unroll
        for (int e = 0; e < 4; ++e) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(w[e], h[e], acc, 0, 0, 0);
    }
};

// G: problems (act step: 1, else train step: 2, with Double DQN 3); NTA: 16-action tiles (1 for A <= 16, else 2).  The leading scalar parameters repeat HeadArgs::partial, rows, A,
// head_blocks, w2[0], b1[0], b2[0] and epsilon: the kernel arguments' first 14 dwords are preloaded into scalar registers when a
// wavefront starts (see conv_tower_kernel); everything else is read from the struct.
template <typename T, int G, int NTA>
__global__ __launch_bounds__(256, sizeof(T) == 4 && G == 3 && NTA == 2 ? 1 : 2) void head_fwd_kernel(const float* partial_, int rows_, int A_, int head_blocks_,
                                                       const void* w2_0_, const float* b1_0_, const float* b2_0_, float epsilon_, HeadArgs a)
{
    typedef HeadMma<T> M;
    typedef typename M::vec V;
    constexpr bool TRAIN = G > 1;
    constexpr int LDH = 512 + 8, STEPS = 128 / M::KS;
    __shared__ __attribute__((aligned(32))) T s_h[G][kHeadRows][LDH];
    __shared__ __attribute__((aligned(16))) float s_red[G][4][kHeadRows][16 * NTA];   // fc2 partial sums: [group][k-quarter wavefront][row][action]
    if constexpr (TRAIN) {
        if (static_cast<int>(blockIdx.x) >= head_blocks_) {
            const int i = static_cast<int>(blockIdx.x) - head_blocks_;
            if (a.desc_out) {
                const int b = i * 256 + static_cast<int>(threadIdx.x);
                if (b < a.gather.B) sample_desc(a.gather, b, a.desc_out + static_cast<size_t>(b) * kDescInts);
            } else gather_block(a.gather, i % 5, i / 5);
            return;
        }
    }
    float h0[4] = {0.f, 0.f, 0.f, 0.f};   // this thread's four features of h (online pass on s)
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int row0 = blockIdx.x * kHeadRows;
    const int lq = lane & 15, kq = lane >> 4;
    const int hr = tid >> 7, hf0 = (tid & 127) * 4;                 // stage (1) and the dzh epilogue: row, features
    const int hrow = row0 + hr < rows_ ? row0 + hr : rows_ - 1;
    const int trow = lane >> 5, tk = lane & 31, tkc = tk < A_ ? tk : A_ - 1;   // tail: row, action of this lane
    const int trow_c = row0 + trow < rows_ ? row0 + trow : rows_ - 1;

    // Every global operand is requested here, before anything waits (a cold round trip to memory costs over a microsecond), in the
    // order in which they are needed, and first those whose addresses came with the wavefront: fc1's slices of ALL groups, fc2's
    // weights, the biases; then what the struct's pointers lead to (a load of them stands in front of every later request).
    const size_t sstride = static_cast<size_t>(rows_) * 512, gstride = sstride * kFc1Slices;
    const float* p0 = partial_ + static_cast<size_t>(hrow) * 512 + hf0;
    float4 v[G][kFc1Slices];
    {   // from a clamped row: no load is ever skipped
#pragma unroll
        for (int g = 0; g < G; ++g)
#pragma unroll
            for (int u = 0; u < kFc1Slices; ++u) v[g][u] = *reinterpret_cast<const float4*>(p0 + g * gstride + u * sstride);
    }
    float4 b1v[G];
    b1v[0] = *reinterpret_cast<const float4*>(b1_0_ + hf0);
    V wf[G][NTA][STEPS];
    auto fetch_w2 = [&](int g, const void* w2) {
#pragma unroll
        for (int ta = 0; ta < NTA; ++ta) {
            const T* wp = static_cast<const T*>(w2) + static_cast<size_t>(min(ta * 16 + lq, A_ - 1)) * 512 + wave * 128 + kq * M::E;
#pragma unroll
            for (int s = 0; s < STEPS; ++s) wf[g][ta][s] = *reinterpret_cast<const V*>(wp + s * M::KS);
        }
    };
    fetch_w2(0, w2_0_);
    float b2_tail[G];
    b2_tail[0] = b2_0_[tkc];
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int g = 1; g < G; ++g) {
        b1v[g] = *reinterpret_cast<const float4*>(a.b1[g] + hf0);
        fetch_w2(g, a.w2[g]);
        b2_tail[g] = a.b2[g][tkc];
    }
    int act_tail = 0;
    float rew_tail = 0.f, done_tail = 0.f;
    bool act_ok = true;   // tail: the stored action of this lane's row lies in [0, A)
    float4 w2row = make_float4(0.f, 0.f, 0.f, 0.f);   // the taken action's row of W2 at this thread's features
    Philox4 draw{};       // act step: the exploration draw of this lane's row
    if constexpr (TRAIN) {
        // A stored action outside [0, A) (replay_sample_gather marks a row it could not assemble with -1) must not
        // address anything: such a row gets loss 0 and gradient 0, and every index derived from it is clamped.
        int act_taken = a.act[hrow];
        act_tail = a.act[trow_c];
        rew_tail = a.rew[trow_c];
        done_tail = a.done[trow_c];
        __builtin_amdgcn_sched_barrier(0);
        act_taken = static_cast<unsigned>(act_taken) < static_cast<unsigned>(A_) ? act_taken : 0;
        act_ok = static_cast<unsigned>(act_tail) < static_cast<unsigned>(A_);
        act_tail = act_ok ? act_tail : 0;
        float w[4];
        load4<T>(static_cast<const T*>(w2_0_) + static_cast<size_t>(act_taken) * 512 + hf0, w);   // used last of all
        w2row = make_float4(w[0], w[1], w[2], w[3]);
    } else {
        draw = philox_draw(a.seed, kTagAct, a.act_step, static_cast<uint32_t>(row0 + trow));
        // computed HERE, under the slices' latency (left alone, the compiler moves the ten rounds into the
        // tail, where only lane 0 of a row uses them and nothing hides them)
        asm volatile("" :: "v"(draw.x[0]), "v"(draw.x[1]));
    }
    __builtin_amdgcn_sched_barrier(0);

    // (1) finish fc1: thread -> (row r = tid / 128, features 4 * (tid % 128) .. + 3), slices added in slice order
    {
        const int row = row0 + hr;
        float4 acc[G];
#pragma unroll
        for (int g = 0; g < G; ++g) acc[g] = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
        for (int g = 0; g < G; ++g)
#pragma unroll
            for (int u = 0; u < kFc1Slices; ++u) { acc[g].x += v[g][u].x; acc[g].y += v[g][u].y; acc[g].z += v[g][u].z; acc[g].w += v[g][u].w; }
#pragma unroll
        for (int g = 0; g < G; ++g) {
            const float4 bv = b1v[g];
            const float4 hv = make_float4(fmaxf(acc[g].x + bv.x, 0.f), fmaxf(acc[g].y + bv.y, 0.f), fmaxf(acc[g].z + bv.z, 0.f),
                                          fmaxf(acc[g].w + bv.w, 0.f));
            store4<T>(&s_h[g][hr][hf0], hv.x, hv.y, hv.z, hv.w);   // a row past the batch repeats the last one; nobody reads its Q
            if (TRAIN && g == 0) {
                h0[0] = hv.x; h0[1] = hv.y; h0[2] = hv.z; h0[3] = hv.w;
                if (row < rows_)
                    store4<T>(static_cast<T*>(a.h_online) + static_cast<size_t>(row) * 512 + hf0, hv.x, hv.y, hv.z, hv.w);
            }
        }
    }
    __syncthreads();
    // (2) fc2: W2 rows (actions) x h columns on the 16x16 instruction; only columns 0 and 1 -- this workgroup's rows -- mean anything
    // (the others repeat them).  The groups' accumulation chains are independent and run side by side; every wavefront's k-quarter
    // goes to LDS, one barrier for all groups.
    {
        f32x4v acc[G][NTA];
#pragma unroll
        for (int g = 0; g < G; ++g)
#pragma unroll
            for (int ta = 0; ta < NTA; ++ta) acc[g][ta] = f32x4v{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int s = 0; s < STEPS; ++s)
#pragma unroll
            for (int g = 0; g < G; ++g) {
                const V hf = *reinterpret_cast<const V*>(&s_h[g][lq & 1][wave * 128 + s * M::KS + kq * M::E]);
#pragma unroll
                for (int ta = 0; ta < NTA; ++ta) M::mma(acc[g][ta], wf[g][ta][s], hf);
            }
        if (lq < kHeadRows) {
#pragma unroll
            for (int g = 0; g < G; ++g)
#pragma unroll
                for (int ta = 0; ta < NTA; ++ta) *reinterpret_cast<f32x4v*>(&s_red[g][wave][lq][ta * 16 + 4 * kq]) = acc[g][ta];
        }
    }
    __syncthreads();

    // Tail: 32 lanes per row (kHeadRows = 2), lane k owns action k.  argmax with the lowest index
    // among equal values (the tie rule of the greedy policy, Section 2.1), as a butterfly over the 32 lanes.
    static_assert(kHeadRows == 2 && kMaxActions <= 32, "tail layout: one wavefront, 32 lanes per row");
    // "Better" is a total order on (value, index), so the pairs may meet in any tree: inside a row of sixteen lanes through
    // the lane-permuting moves of the vector unit (neighbours, pairs, mirrored halves of eight, mirrored sixteen -- a few
    // cycles each), across the two sixteens through one cross-lane exchange (ten of those in a row were 0.6 us of a 3 us kernel).
    auto argmax_lowest = [&](float v, int k) {   // lanes 0 .. 15 of the row return the winner
        int best = k;
        auto meet = [&](float ov, int ob) {
            if (ov > v || (ov == v && ob < best)) { v = ov; best = ob; }
        };
#define DQN_ARGMAX_DPP(ctrl)                                                                                              \
        meet(__builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), ctrl, 0xF, 0xF, false)), \
             __builtin_amdgcn_update_dpp(0, best, ctrl, 0xF, 0xF, false))
        DQN_ARGMAX_DPP(0xB1);    // quad_perm [1, 0, 3, 2]: lane ^ 1
        DQN_ARGMAX_DPP(0x4E);    // quad_perm [2, 3, 0, 1]: lane ^ 2
        DQN_ARGMAX_DPP(0x141);   // row_half_mirror: lane i of eight <-> 7 - i (the other quad)
        DQN_ARGMAX_DPP(0x140);   // row_mirror: lane i of sixteen <-> 15 - i (the other eight)
#undef DQN_ARGMAX_DPP
        // the other sixteen of the row: its result is read from its first lane (16, or 48 for the second row) -- a scalar
        // broadcast, where a cross-lane exchange costs ten times as much.  Only the FIRST sixteen lanes of a row end up with
        // the row's winner; the callers use lane 0 of the row.
        const int hv = lane < 32 ? __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), 16) : __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), 48);
        const int hb = lane < 32 ? __builtin_amdgcn_readlane(best, 16) : __builtin_amdgcn_readlane(best, 48);
        meet(__builtin_bit_cast(float, hv), hb);
        return best;
    };
    const float kNegInf = -__builtin_huge_valf();
    // Q_g(row trow, action tk): the four k-quarter partials are added in wavefront order, then the bias
    auto q_of = [&](int g) { return (((s_red[g][0][trow][tkc] + s_red[g][1][trow][tkc]) + s_red[g][2][trow][tkc]) + s_red[g][3][trow][tkc]) + b2_tail[g]; };
    if constexpr (!TRAIN) {
        if (wave != 0) return;
        const int row = row0 + trow;
        const float qv = tk < A_ ? q_of(0) : kNegInf;
        int act = argmax_lowest(qv, tk);
        if (row >= rows_) return;
        if (a.q_out && tk < A_) a.q_out[static_cast<size_t>(row) * A_ + tk] = qv;
        if (tk == 0) {
            const Philox4 d = draw;
            const float u = static_cast<float>(d.x[0] >> 8) * 0x1p-24f;
            if (u < epsilon_) act = static_cast<int>((static_cast<uint64_t>(d.x[1]) * static_cast<uint32_t>(A_)) >> 32);
            a.actions[row] = act;
        }
    } else {
        __shared__ float s_dq[kHeadRows];
        if (wave == 0) {
            const float q0 = q_of(0), q1 = q_of(1);
            const float q2 = G > 2 ? q_of(G - 1) : 0.f;   // Double DQN: Q(s', .; theta) selects the action
            const int astar = argmax_lowest(tk < A_ ? (G > 2 ? q2 : q1) : kNegInf, tk);
            const int row = row0 + trow;
            const bool live = row < rows_;
            if (live && tk < A_) {
                float* q = a.q_all + static_cast<size_t>(row) * A_ + tk;
                const size_t gs = static_cast<size_t>(rows_) * A_;
                q[0] = q0;
                q[gs] = q1;
                if (G > 2) q[2 * gs] = q2;
            }
            // the two values the TD error needs sit in other lanes of this row: Q(s', a*; theta^-) and Q(s, a_b; theta)
            const float q1_star = __shfl(q1, astar, 32), q0_taken = __shfl(q0, act_tail, 32);
            if (tk == 0) {
                const float y = rew_tail + a.gamma * (1.f - done_tail) * q1_star;
                const float delta = q0_taken - y, ad = fabsf(delta);
                const float loss = act_ok ? (ad <= a.huber ? 0.5f * delta * delta : a.huber * (ad - 0.5f * a.huber)) : 0.f;
                const float dq = act_ok ? fminf(fmaxf(delta, -a.huber), a.huber) / static_cast<float>(rows_) : 0.f;
                s_dq[trow] = dq;
                if (live) { a.lossv[row] = loss; a.dqv[row] = dq; }
            }
        }
        __syncthreads();
        // fc2's data gradient through fc1's ReLU for this workgroup's rows: dQ has one non-zero per row
        const int row = row0 + hr;
        if (row < rows_) {
            const float dq = s_dq[hr];
            store4<T>(static_cast<T*>(a.dzh) + static_cast<size_t>(row) * 512 + hf0, h0[0] > 0.f ? dq * w2row.x : 0.f,
                      h0[1] > 0.f ? dq * w2row.y : 0.f, h0[2] > 0.f ? dq * w2row.z : 0.f, h0[3] > 0.f ? dq * w2row.w : 0.f);
        }
    }
}

// Small reductions of the backward pass, one launch:
//  * blocks [0, bias_blocks): fc1's bias gradient = column sums of dzh ([B][512], T), first stage: a block sums kFc1BiasRows rows into
//    partial[block][512]; the optimiser kernel adds the chunks in order, so no atomics and no extra launch are needed (the conv
//    layers' bias gradients come out of their weight-gradient workgroups, where dZ is in LDS);
//  * the last 33 blocks: fc2's weight gradient (32 blocks of 16 columns) and its bias gradient + loss.  dQ has one non-zero per row (the taken action):
//    dW2[a][o] = sum_{b: a_b = a} dq_b h[b][o];  db2[a] = sum_{b: a_b = a} dq_b;  loss = mean_b loss_b.
//    Each block owns 16 columns o; thread (o, part) accumulates the samples b = part (mod 16) in
//    increasing order into its own LDS column, the sixteen parts are then added in order.
constexpr int kFc1BiasRows = 64;   // a workgroup covers four rows per pass: one round trip of 16 loads in flight
// The optimiser's conv blocks: lanes per four weights, slices per lane and round trip (64 of conv1's at most 128 slices in flight, 48
// of the at most 44 -- fp32: 64 -- of the others).
constexpr int kRmsLanes1 = 8, kRmsTrip1 = 8, kRmsLanes23 = 4, kRmsTrip23 = 12;
constexpr int kRmsQuads1 = 32 * 256 / 4, kRmsQuads2 = 64 * 512 / 4, kRmsQuads3 = 64 * 576 / 4;
constexpr int kRmsBlocks1 = kRmsQuads1 * kRmsLanes1 / 256, kRmsBlocks2 = kRmsQuads2 * kRmsLanes23 / 256, kRmsBlocks3 = kRmsQuads3 * kRmsLanes23 / 256;
constexpr int kRmsConvBlocks = kRmsBlocks1 + kRmsBlocks2 + kRmsBlocks3;   // 64 + 128 + 144
static_assert(kRmsBlocks1 * 256 == kRmsQuads1 * kRmsLanes1 && kRmsBlocks2 * 256 == kRmsQuads2 * kRmsLanes23 && kRmsBlocks3 * 256 == kRmsQuads3 * kRmsLanes23, "whole blocks");
constexpr int kRmsFc1Tiles = 8 * 49;                                // 64 x 64 tiles of fc1.w
// Split-K slices of the conv weight gradients, [slice][tensor] fp32 for each layer, in one buffer (conv1's gradient is small: more
// slices are cheap).
constexpr size_t kWgMaxSplits = 64, kWgMaxSplits1 = 128;
constexpr size_t kWgOff1 = 0, kWgOff2 = kWgMaxSplits1 * 32 * 256, kWgOff3 = kWgOff2 + kWgMaxSplits * 64 * 512;
constexpr size_t kWgTotal = kWgOff3 + kWgMaxSplits * 64 * 576;
constexpr int kRmsBiasLanes = 8;                                    // lanes per channel in the optimiser's bias blocks
constexpr int kRmsBiasBlocks = (672 * kRmsBiasLanes + 255) / 256;  // 32 + 64 + 64 + 512 hidden-layer bias channels
struct BiasGradArgs {
    const void* dzh;        // T [B][512]
    int bias_blocks;
    float* partial;         // [bias_blocks][512]
    // fc2 weight gradient
    const void* h;          // T [B][512]
    const int32_t* act;
    const float* dqv;
    const float* lossv;
    int B, A;
    float* g_w2;
    float* g_b2;
    float* loss_out;
    float* loss_keep;
};
constexpr size_t kSmallGradsSmem = (256 * 9 + kMaxBatch) * sizeof(float) + kMaxBatch * sizeof(int) + kMaxActions * 256 * sizeof(float);
constexpr int kSmallGradsExtraBlocks = 33;   // fc2 weight gradient (32) + fc2 bias gradient / loss (1)

// One workgroup of the small reductions; `block` counts from the first bias block, smem holds
// kSmallGradsSmem bytes.
template <typename T>
__device__ inline void small_grads_block(const BiasGradArgs& args, int block, unsigned char* smem)
{
    typedef typename Vec8<T>::type V8;
    float (*red)[9] = reinterpret_cast<float (*)[9]>(smem);
    float* s_dq = reinterpret_cast<float*>(smem) + 256 * 9;
    int* s_a = reinterpret_cast<int*>(s_dq + kMaxBatch);
    float (*s_acc)[256] = reinterpret_cast<float (*)[256]>(s_a + kMaxBatch);
    const int tid = threadIdx.x;
    if (block >= args.bias_blocks) {
        const int B = args.B, A = args.A;
        const T* h = static_cast<const T*>(args.h);
        float* s_loss = &red[0][0];   // 256 * 9 floats: room for kMaxBatch loss terms
        for (int b = tid; b < B; b += 256) {
            // a row whose stored action lies outside [0, A) has dq = 0 (head kernel); its index must still not leave s_acc
            const int ab = args.act[b];
            const bool ok = static_cast<unsigned>(ab) < static_cast<unsigned>(A);
            s_dq[b] = ok ? args.dqv[b] : 0.f; s_a[b] = ok ? ab : 0; s_loss[b] = args.lossv[b];
        }
        for (int a = 0; a < A; ++a) s_acc[a][tid] = 0.f;
        __syncthreads();
        // 16 columns per block; thread (o, part): samples b = part (mod 16) in increasing order.
        // Block 32 is the bias "column" (h = 1) and also owns the batch-mean loss.
        const int ob = block - args.bias_blocks;
        const int oo = tid & 15, part = tid >> 4;
        const bool bias_block = ob == 32;
        const int o = ob * 16 + oo;
        // sixteen samples in flight per thread (clamped address: no load is ever skipped)
        const size_t oc = bias_block ? 0 : o;
        for (int b0 = part; b0 < B; b0 += 256) {
            T hv[16];
#pragma unroll
            for (int u = 0; u < 16; ++u) {
                const int b = b0 + 16 * u;
                hv[u] = h[static_cast<size_t>(b < B ? b : B - 1) * 512 + oc];
            }
#pragma unroll
            for (int u = 0; u < 16; ++u) {
                const int b = b0 + 16 * u;
                if (b < B) s_acc[s_a[b]][tid] += s_dq[b] * (bias_block ? 1.f : to_float(hv[u]));
            }
        }
        __syncthreads();
        for (int a = part; a < A; a += 16) {
            float sum = 0.f;
#pragma unroll
            for (int p = 0; p < 16; ++p) sum += s_acc[a][p * 16 + oo];
            if (!bias_block) args.g_w2[static_cast<size_t>(a) * 512 + o] = sum;
            else if (oo == 0) args.g_b2[a] = sum;
        }
        if (bias_block) {
            // loss = (1/B) sum_b loss_b: thread t adds b = t, t+256, .. then a fixed binary tree
            __syncthreads();
            float acc = 0.f;
            for (int b = tid; b < B; b += 256) acc += s_loss[b];
            __syncthreads();
            s_loss[tid] = acc;
            __syncthreads();
            for (int stride = 128; stride >= 1; stride >>= 1) {
                if (tid < stride) s_loss[tid] += s_loss[tid + stride];
                __syncthreads();
            }
            if (tid == 0) {
                const float mean = s_loss[0] / static_cast<float>(B);
                *args.loss_keep = mean;
                if (args.loss_out) *args.loss_out = mean;
            }
        }
        return;
    }
    // column sums of one chunk of rows, all channels: thread -> (16-byte vector of the row, row mod RP), so a
    // pass of the workgroup reads RP whole rows, fully coalesced; the RP partial rows meet in LDS in row order
    constexpr int C = 512, VR = C / 8, RP = 256 / VR;
    static_assert(RP == 4, "four lanes per channel add the partial rows");
    const int vec = tid % VR, rsub = tid / VR;
    const T* dz = static_cast<const T*>(args.dzh) + vec * 8;
    const int r_end = min(args.B, (block + 1) * kFc1BiasRows);
    float acc[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) acc[e] = 0.f;
    // sixteen rows in flight per thread (clamped address, masked value: no load is ever skipped)
    static_assert(16 * RP == kFc1BiasRows, "one pass");
    {
        const int r = block * kFc1BiasRows + rsub;
        V8 v[16];
#pragma unroll
        for (int u = 0; u < 16; ++u) {
            const int rr = r + u * RP;
            v[u] = vec8_keep<T>(*reinterpret_cast<const V8*>(dz + static_cast<size_t>(rr < r_end ? rr : r_end - 1) * C), rr < r_end);
        }
#pragma unroll
        for (int u = 0; u < 16; ++u)
#pragma unroll
            for (int e = 0; e < 8; ++e) acc[e] += to_float(v[u][e]);
    }
#pragma unroll
    for (int e = 0; e < 8; ++e) red[tid][e] = acc[e];
    __syncthreads();
    // four lanes per channel hold one partial row each and meet in a fixed tree
    for (int i = tid; i < 4 * C; i += 256) {
        const int c = i >> 2, j = i & 3;
        float sum = red[j * VR + (c >> 3)][c & 7];
        sum += __shfl_down(sum, 2, 4);
        sum += __shfl_down(sum, 1, 4);
        if (j == 0) args.partial[static_cast<size_t>(block) * C + c] = sum;
    }
}

// ---- optimiser --------------------------------------------------------------------------------

struct RmsArgs {
    float* theta;
    float* grad;
    float* v;
    float* m;
    void* sh;        // forward operand copy
    void* bsh;       // backward operand copies
    Offsets off;
    float lr, alpha, eps;
    int centered;
    // second stage of the bias gradients (conv1..3, fc1): chunk sums (conv layers: one per weight-gradient slice)
    const float* bias_partial;   // (full precision: conv layers fp64)
    int bias_chunks[4];
    int bias_first[4];           // in floats
};

__device__ inline void rms_update(const RmsArgs& a, float& th, float g, float& vv, float& mm)
{
    vv = a.alpha * vv + (1.f - a.alpha) * g * g;
    float var = vv;
    if (a.centered) {
        mm = a.alpha * mm + (1.f - a.alpha) * g;
        var = fmaxf(vv - mm * mm, 0.f);
    }
    th -= a.lr * g / (sqrtf(var) + a.eps);
}

// Conv weights of layer CONV: the gradient arrives as `ns` split-K slices.  LANES adjacent lanes share four weights: lane j requests
// slices j, j + LANES, ... (TRIP per round trip), the sums meet in a fixed tree, lanes 0 .. 3 update one
// weight each.  Whatever LANES is, there are eight sums (every eighth slice, in order) and one tree, so that the number of lanes
// does not show in the gradient's bits: four lanes keep two sums each.  What counts is the length of the dependent chain: everything an address needs is a constant or comes with the
// wavefront, and the parameters are requested with the slices.  (Offsets and counts read from the argument struct, one lane updating
// all four weights and eight lanes per quad everywhere: these blocks alone were a launch of 8.1 us, now 4.2 us, and the whole
// kernel 10.7 / 12.1 us at batch 32 / 256, now 9.2 / 10.5 us, back to back.)
template <typename T, int CONV, int LANES, int TRIP>
__device__ inline void rms_conv_block(float* theta, float* grad, float* v, float* m, const float* slices, int ns, const RmsArgs& a, int block)
{
    constexpr size_t E0 = CONV == 0 ? kOffW1 : CONV == 1 ? kOffW2 : kOffW3, TSIZE = CONV == 0 ? 32 * 256 : CONV == 1 ? 64 * 512 : 64 * 576;
    const int idx = block * 256 + static_cast<int>(threadIdx.x), j = idx % LANES;
    const int r = idx / LANES * 4;
    const float* p = slices + (CONV == 0 ? kWgOff1 : CONV == 1 ? kWgOff2 : kWgOff3) + r;
    const size_t e = E0 + r + (j & 3);
    float4 v4[TRIP];
#pragma unroll
    for (int u = 0; u < TRIP; ++u) v4[u] = *reinterpret_cast<const float4*>(p + static_cast<size_t>(min(j + u * LANES, ns - 1)) * TSIZE);
    float th = theta[e], vv = v[e], mm = m[e];
    __builtin_amdgcn_sched_barrier(0);
    constexpr int SUMS = 8 / LANES;
    static_assert(SUMS * LANES == 8 && TRIP % SUMS == 0, "eight sums, whichever lanes hold them");
    float4 part[SUMS];
#pragma unroll
    for (int k = 0; k < SUMS; ++k) part[k] = make_float4(0.f, 0.f, 0.f, 0.f);
    for (int s0 = j; s0 < ns; s0 += TRIP * LANES) {
#pragma unroll
        for (int u = 0; u < TRIP; ++u)
            if (s0 + u * LANES < ns) { float4& to = part[u % SUMS]; to.x += v4[u].x; to.y += v4[u].y; to.z += v4[u].z; to.w += v4[u].w; }
        if (s0 + TRIP * LANES < ns) {
#pragma unroll
            for (int u = 0; u < TRIP; ++u) v4[u] = *reinterpret_cast<const float4*>(p + static_cast<size_t>(min(s0 + (TRIP + u) * LANES, ns - 1)) * TSIZE);
        }
    }
    float4 sum = part[0];
    if (SUMS == 2) { sum.x += part[SUMS - 1].x; sum.y += part[SUMS - 1].y; sum.z += part[SUMS - 1].z; sum.w += part[SUMS - 1].w; }
#pragma unroll
    for (int d = LANES / 2; d >= 1; d >>= 1) {
        sum.x += __shfl_xor(sum.x, d, LANES); sum.y += __shfl_xor(sum.y, d, LANES);
        sum.z += __shfl_xor(sum.z, d, LANES); sum.w += __shfl_xor(sum.w, d, LANES);
    }
    if (j >= 4) return;
    float g = j == 0 ? sum.x : j == 1 ? sum.y : j == 2 ? sum.z : sum.w;
    if (CONV == 0) g *= 1.f / 255.f;
    grad[e] = g;
    rms_update(a, th, g, vv, mm);
    theta[e] = th;
    v[e] = vv;
    if (a.centered) m[e] = mm;
    const int el = r + j;
    if (CONV == 0) {
        if (sizeof(T) == 2) reinterpret_cast<_Float16*>(a.sh)[tower_frag_index(el / 256, el % 256, 256)] = static_cast<_Float16>(th);
        else static_cast<T*>(a.sh)[el] = from_float<T>(th);
    } else {
        constexpr int K = CONV == 1 ? 512 : 576;
        if (sizeof(T) == 2) static_cast<T*>(a.sh)[E0 + tower_frag_index(el / K, el % K, K)] = from_float<T>(th);
        else store_thirds(reinterpret_cast<bf16_t*>(static_cast<T*>(a.sh) + thirds_offset(a.off)) + (CONV == 1 ? kThirdsW2 : kThirdsW3), el / K, el % K, K, th);
        if (CONV == 1) bsh_store_w2<T>(static_cast<T*>(a.bsh), el, th); else bsh_store_w3<T>(static_cast<T*>(a.bsh), el, th);
    }
}

// Centered RMSProp (Appendix B) fused with the refresh of the operand copies.  The conv weights' blocks come first (a dependent chain);
// fc1.w (95 % of the parameters) is walked in 64 x 64 tiles whose two operand copies (forward [o][f] and backward [f][o], both in
// fragment order) are written in whole 512-byte pieces via LDS; then fc2 element by element and the hidden-layer biases.  Bound by memory traffic (62 MB at batch 32: 6.8
// TB/s back to back).
// The leading scalar parameters repeat RmsArgs' pointers and what the blocks need before their first load (splits: slices per conv
// layer, one byte each): the kernel arguments' first 14 dwords are preloaded into scalar registers when a wavefront starts (see
// conv_tower_kernel).
template <typename T>
__global__ __launch_bounds__(256) void rmsprop_kernel(float* theta_, float* grad_, float* v_, float* m_, const float* slices_, uint32_t splits_, int flat_blocks_, RmsArgs a)
{
    __shared__ T tile[64][64 + 8];   // [f][o]
    const int tid = threadIdx.x;
    int block = static_cast<int>(blockIdx.x);
    if (block < kRmsConvBlocks) {
        if (block < kRmsBlocks1) rms_conv_block<T, 0, kRmsLanes1, kRmsTrip1>(theta_, grad_, v_, m_, slices_, splits_ & 255, a, block);
        else if (block < kRmsBlocks1 + kRmsBlocks2)
            rms_conv_block<T, 1, kRmsLanes23, kRmsTrip23>(theta_, grad_, v_, m_, slices_, (splits_ >> 8) & 255, a, block - kRmsBlocks1);
        else rms_conv_block<T, 2, kRmsLanes23, kRmsTrip23>(theta_, grad_, v_, m_, slices_, (splits_ >> 16) & 255, a, block - kRmsBlocks1 - kRmsBlocks2);
        return;
    }
    block -= kRmsConvBlocks;
    if (block < kRmsFc1Tiles) {   // rows o0 .. o0+63, columns f0 .. f0+63; a thread's sixteen parameters are in flight at once
        const int o0 = (block / 49) * 64, f0 = (block % 49) * 64;
        const int r0 = tid / 16, c4 = (tid % 16) * 4;
        float4 th[4], g[4], vv[4], mm[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const size_t e = kOffWf1 + static_cast<size_t>(o0 + r0 + 16 * u) * 3136 + f0 + c4;
            th[u] = *reinterpret_cast<float4*>(theta_ + e);
            g[u] = *reinterpret_cast<const float4*>(grad_ + e);
            vv[u] = *reinterpret_cast<float4*>(v_ + e);
            mm[u] = *reinterpret_cast<float4*>(m_ + e);
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int r = r0 + 16 * u;
            const size_t e = kOffWf1 + static_cast<size_t>(o0 + r) * 3136 + f0 + c4;
            rms_update(a, th[u].x, g[u].x, vv[u].x, mm[u].x);
            rms_update(a, th[u].y, g[u].y, vv[u].y, mm[u].y);
            rms_update(a, th[u].z, g[u].z, vv[u].z, mm[u].z);
            rms_update(a, th[u].w, g[u].w, vv[u].w, mm[u].w);
            *reinterpret_cast<float4*>(theta_ + e) = th[u];
            *reinterpret_cast<float4*>(v_ + e) = vv[u];
            if (a.centered) *reinterpret_cast<float4*>(m_ + e) = mm[u];
            tile[c4 + 0][r] = from_float<T>(th[u].x);
            tile[c4 + 1][r] = from_float<T>(th[u].y);
            tile[c4 + 2][r] = from_float<T>(th[u].z);
            tile[c4 + 3][r] = from_float<T>(th[u].w);
        }
        __syncthreads();
        // pieces of 32 rows x 16 bytes of consecutive k, one per 32 threads
        constexpr int E = 16 / static_cast<int>(sizeof(T)), PIECES = 64 * 64 / (32 * E), KP = 64 / E;
        typedef T vec __attribute__((ext_vector_type(16 / sizeof(T))));
        const int rr = tid & 31;
#pragma unroll
        for (int u = 0; u < PIECES / 8; ++u) {
            const int piece = (tid >> 5) + 8 * u, row = piece / KP * 32 + rr, k = piece % KP * E;
            *reinterpret_cast<vec*>(static_cast<T*>(a.bsh) + bsh_index_wf1<T>(o0 + k, f0 + row)) = *reinterpret_cast<const vec*>(&tile[row][k]);   // rows f, k = o
            vec val;                                                                                                                         // rows o, k = f
#pragma unroll
            for (int j = 0; j < E; ++j) val[j] = tile[k + j][row];
            *reinterpret_cast<vec*>(static_cast<T*>(a.sh) + kOffWf1 + frag_index<T>(o0 + row, f0 + k, 3136)) = val;
        }
        return;
    }
    block -= kRmsFc1Tiles;
    if (block < flat_blocks_) {
        const size_t n = a.off.total - kOffWf2, n4 = n / 4;   // fc2's weights and biases: the end of the blob, 4-aligned
        const size_t i = block * static_cast<size_t>(256) + tid;
        if (i < n4) {
            const size_t e = kOffWf2 + 4 * i;
            float4 th = *reinterpret_cast<float4*>(theta_ + e);
            const float4 g = *reinterpret_cast<const float4*>(grad_ + e);
            float4 vv = *reinterpret_cast<float4*>(v_ + e);
            float4 mm = *reinterpret_cast<float4*>(m_ + e);
            rms_update(a, th.x, g.x, vv.x, mm.x);
            rms_update(a, th.y, g.y, vv.y, mm.y);
            rms_update(a, th.z, g.z, vv.z, mm.z);
            rms_update(a, th.w, g.w, vv.w, mm.w);
            *reinterpret_cast<float4*>(theta_ + e) = th;
            *reinterpret_cast<float4*>(v_ + e) = vv;
            if (a.centered) *reinterpret_cast<float4*>(m_ + e) = mm;
            store4<T>(static_cast<T*>(a.sh) + e, th.x, th.y, th.z, th.w);
        } else if (i < n4 + (n - 4 * n4)) {
            const size_t e = kOffWf2 + 4 * n4 + (i - n4);
            float th = theta_[e], vv = v_[e], mm = m_[e];
            rms_update(a, th, grad_[e], vv, mm);
            theta_[e] = th;
            v_[e] = vv;
            if (a.centered) m_[e] = mm;
            static_cast<T*>(a.sh)[e] = from_float<T>(th);
        }
        return;
    }
    {
        // hidden-layer biases: finish the gradient, then update.  Eight adjacent lanes share a channel: lane j
        // adds chunks j, j + 8, ... in order, then the eight sums meet in a fixed tree -- a large batch has
        // hundreds of chunks and one lane walking them alone was the tail of this kernel.
        const int idx = (block - flat_blocks_) * 256 + tid;
        const int ch = idx / kRmsBiasLanes, j = idx % kRmsBiasLanes;
        const bool live = ch < 32 + 64 + 64 + 512;
        int layer = 3, c = 0;
        size_t e = 0;
        if (ch < 32) { layer = 0; c = ch; e = a.off.b1 + c; }
        else if (ch < 96) { layer = 1; c = ch - 32; e = a.off.b2 + c; }
        else if (ch < 160) { layer = 2; c = ch - 96; e = a.off.b3 + c; }
        else if (live) { layer = 3; c = ch - 160; e = a.off.bf1 + c; }
        const int C = layer == 0 ? 32 : (layer == 3 ? 512 : 64);
        const float* part = a.bias_partial + a.bias_first[layer];
        typedef typename std::conditional<sizeof(T) == 4, double, float>::type Sum;   // full precision: the conv layers' partials are fp64
        Sum total = 0;
        if (live)
            for (int k = j; k < a.bias_chunks[layer]; k += kRmsBiasLanes)
                total += layer < 3 ? reinterpret_cast<const Sum*>(part)[k * C + c] : part[k * C + c];
        total += __shfl_down(total, 4, kRmsBiasLanes);
        total += __shfl_down(total, 2, kRmsBiasLanes);
        total += __shfl_down(total, 1, kRmsBiasLanes);
        if (!live || j != 0) return;
        const float g = static_cast<float>(total);
        grad_[e] = g;
        float th = theta_[e], vv = v_[e], mm = m_[e];
        rms_update(a, th, g, vv, mm);
        theta_[e] = th;
        v_[e] = vv;
        if (a.centered) m_[e] = mm;
        static_cast<T*>(a.sh)[e] = from_float<T>(th);
        return;
    }
}

// Builds every operand copy of theta from the fp32 master (after dqn_set_params).
template <typename T>
__global__ __launch_bounds__(256) void build_copies_kernel(const float* __restrict__ theta, T* __restrict__ sh,
                                                           T* __restrict__ bsh, Offsets off)
{
    const size_t e = blockIdx.x * static_cast<size_t>(blockDim.x) + threadIdx.x;
    if (e >= off.total) return;
    const T val = from_float<T>(theta[e]);
    shadow_store<T>(sh, off, e, theta[e]);
    if (bsh) {
        if (e >= off.w2 && e < off.b2) bsh_store_w2<T>(bsh, static_cast<int>(e - off.w2), theta[e]);
        else if (e >= off.w3 && e < off.b3) bsh_store_w3<T>(bsh, static_cast<int>(e - off.w3), theta[e]);
        else if (e >= off.wf1 && e < off.bf1) {
            const size_t r = e - off.wf1;
            bsh[bsh_index_wf1<T>(static_cast<int>(r / 3136), static_cast<int>(r % 3136))] = val;
        }
    }
}

// theta^- <- theta: fp32 master (bitwise) and the forward operand copy.
template <typename T>
__global__ __launch_bounds__(256) void target_copy_kernel(const float* __restrict__ theta, float* __restrict__ theta_t,
                                                          const T* __restrict__ sh, T* __restrict__ sh_t, size_t n, size_t n_copy)
{
    const size_t i = blockIdx.x * static_cast<size_t>(blockDim.x) + threadIdx.x;
    if (i < n) theta_t[i] = theta[i];
    if (i < n_copy) sh_t[i] = sh[i];
}

}  // namespace dqn
