// Units cut into slices (device side; the host's rule is in apar_pool.cpp).
//
// A launch whose heaviest units are more than a compute unit's share of the work ends on them while the rest of the
// chip idles - a call with few threads has nothing but such units, and its wavefronts walk their lists at one tile
// per memory latency.  Such units are launched as several workgroups: slice s of n takes the part
// [len * s / n, len * (s + 1) / n) of each of the unit's tile lists (attention is a set operation over the blocks).
// Every wavefront leaves its rows' states in `state`, and the last of a unit's slices to arrive - per wavefront,
// counted in `arrived` - folds them, in slice order, so that the result does not depend on who came last.  Nobody
// waits for anybody.  `arrived` is zero before a launch and after it.
#pragma once

#include <hip/hip_runtime.h>

#include "apar_internal.hpp"

namespace apar {

struct Slice {
    int wg = 0;        // workgroup descriptor
    int s = 0, n = 1;  // this slice of n
    int state = 0, cut = 0;
};

// blockIdx.x -> unit and slice (kv heads fastest).
__device__ __forceinline__ Slice slice_of_block(const SplitPlan& sp, int first, int n_kv) {
    const SplitBlock b = sp.blocks[first + blockIdx.x / n_kv];
    Slice r;
    r.wg = b.wg;
    r.s = b.slice & 0xffff;
    r.n = b.slice >> 16;
    r.state = b.state;
    r.cut = b.cut;
    return r;
}

// The slice's part of a list of n tiles whose first n_full are full.
__device__ __forceinline__ void cut_list(const Slice& sl, int& ofs, int& n, int& n_full) {
    const int b = (int)((int64_t)n * sl.s / sl.n), e = (int)((int64_t)n * (sl.s + 1) / sl.n);
    ofs += b;
    n = e - b;
    n_full = max(0, min(e, n_full) - b);
}

// Leaves this wavefront's row states (NT tiles of J x 4 accumulators, reference and share of the sum per lane) and, in
// the last slice of the unit to come here, replaces them by the states over the whole unit.  Returns whether this
// wavefront goes on to write the rows.  wave, n_waves: this wavefront among those of the workgroup that leave states.
// JT > J: the wavefronts of a workgroup hold J of one tile's JT accumulators each, from j0 on, and the same references and sums;
// n_waves is 1 then (they leave one state together), and each of them folds its own part.
template <int NT, int J, int JT = J, class State>
__device__ __forceinline__ bool fold_slices(const SplitPlan& sp, const Slice& sl, int n_kv, int kvh, int wave, int n_waves, int lane,
                                            State (&st)[NT], int j0 = 0) {
    typedef __attribute__((__vector_size__(4 * sizeof(float)))) float f32x4;
    typedef __attribute__((__vector_size__(2 * sizeof(float)))) float f32x2;
    typedef __attribute__((__vector_size__(4 * sizeof(uint32_t)))) uint32_t u32x4;
    typedef __attribute__((__vector_size__(2 * sizeof(uint32_t)))) uint32_t u32x2;
    if (sl.n == 1) return true;
    constexpr int kTileBytes = (JT * 4 + 2) * 64 * 4;
    // The states go past the L2 of this XCD (sc1: agent scope) and are read back the same way: what a release and an
    // acquire fence of agent scope would do instead - write back and invalidate the whole L2, per wavefront - costs
    // more than the slices gain (one request of 4 threads, 32 heads, 512 workgroups: 33 us with fences, 23 us without).
    constexpr int kAgent = 16;
    const __amdgpu_buffer_rsrc_t state = __builtin_amdgcn_make_buffer_rsrc(sp.state, 0, (int)kSplitStateBytes, 0x00027000);
    const int step = n_waves * NT * kTileBytes;  // from one slice to the next
    const int base = (sl.state * n_kv + (kvh * sl.n * n_waves + (JT > J ? 0 : wave)) * NT) * kTileBytes;
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
        const int at = base + sl.s * step + nt * kTileBytes;
#pragma unroll
        for (int jj = 0; jj < J; ++jj)
            __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, st[nt].o[jj]), state, at + ((j0 + jj) * 64 + lane) * 16, 0, kAgent);
        __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2, f32x2{st[nt].m, st[nt].l}), state, at + JT * 1024 + lane * 8, 0, kAgent);
    }
    int32_t* counter = sp.arrived + (sl.cut * n_kv + kvh) * 4 + wave;
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // the states have arrived before the count says so
    int before = 0;
    if (lane == 0) before = __hip_atomic_fetch_add(counter, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (__builtin_amdgcn_readfirstlane(before) != sl.n - 1) return false;
    asm volatile("" ::: "memory");
    if (lane == 0) __hip_atomic_store(counter, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
        const int at = base + nt * kTileBytes;
        // One pass, the reference moving along (a pass for the largest one first is another latency per slice), three
        // slices in flight.  Against two passes and two slices: one request, 8 kv heads, 2 k - 8 k tokens 14.4 -> 11.9 us,
        // 9 k - 30 k tokens 33.8 -> 29.7, 12 threads 15.4 -> 14.7.
        float m = -INFINITY;
        float l = 0.0f;
        f32x4 o[J];
#pragma unroll
        for (int jj = 0; jj < J; ++jj) o[jj] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
        if constexpr (JT > J) {
            // a quarter of a state per wavefront: eight slices in flight (one thread family of 6 k to 22 k tokens on an fp8 pool, 4 kv heads,
            // 48 slices: 24.0 -> 21.7 us, with one 32 k long and 8 kv heads 32.6 -> 30.6)
            constexpr int kAhead = 8;
            for (int s0 = 0; s0 < sl.n; s0 += kAhead) {
                f32x2 ml[kAhead];
                f32x4 os[kAhead][J];
#pragma unroll
                for (int i = 0; i < kAhead; ++i)
                    ml[i] = __builtin_bit_cast(f32x2, __builtin_amdgcn_raw_buffer_load_b64(state, at + min(s0 + i, sl.n - 1) * step + JT * 1024 + lane * 8, 0, kAgent));
#pragma unroll
                for (int i = 0; i < kAhead; ++i) {
                    // Past the last slice: past the descriptor's end, where a buffer load gives zeros.  (Not the last slice again, whose
                    // infinities a weight of 0 would make NaN.)
                    const int as = at + (s0 + i) * step + (((sl.n - 1 - s0 - i) >> 31) & (int)kSplitStateBytes);
#pragma unroll
                    for (int jj = 0; jj < J; ++jj)
                        os[i][jj] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(state, as + ((j0 + jj) * 64 + lane) * 16, 0, kAgent));
                }
                float mx = m;  // (of slices that are read twice too)
#pragma unroll
                for (int i = 0; i < kAhead; ++i) mx = fmaxf(mx, ml[i][0]);
                const float a = mx == -INFINITY ? 1.0f : __builtin_amdgcn_exp2f(m - mx);
                l *= a;
#pragma unroll
                for (int jj = 0; jj < J; ++jj) o[jj] *= a;
#pragma unroll
                for (int i = 0; i < kAhead; ++i) {
                    // (a slice that saw nothing of the row left m = -inf and zeros; past the last slice: nothing)
                    const float b = (s0 + i < sl.n) & (ml[i][0] != -INFINITY) ? __builtin_amdgcn_exp2f(ml[i][0] - mx) : 0.0f;
                    l += b * ml[i][1];
#pragma unroll
                    for (int jj = 0; jj < J; ++jj) o[jj] += b * os[i][jj];
                }
                m = mx;
            }
        } else {
#pragma unroll(3)
            for (int s = 0; s < sl.n; ++s) {
                const int as = at + s * step;
                const f32x2 ml = __builtin_bit_cast(f32x2, __builtin_amdgcn_raw_buffer_load_b64(state, as + JT * 1024 + lane * 8, 0, kAgent));
                f32x4 os[J];
#pragma unroll
                for (int jj = 0; jj < J; ++jj)
                    os[jj] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(state, as + ((j0 + jj) * 64 + lane) * 16, 0, kAgent));
                // (a slice that saw nothing of the row left m = -inf and zeros)
                const float mx = fmaxf(m, ml[0]);
                const float a = mx == -INFINITY ? 1.0f : __builtin_amdgcn_exp2f(m - mx);
                const float b = mx == -INFINITY ? 1.0f : __builtin_amdgcn_exp2f(ml[0] - mx);
                l = a * l + b * ml[1];
#pragma unroll
                for (int jj = 0; jj < J; ++jj) o[jj] = a * o[jj] + b * os[jj];
                m = mx;
            }
        }
        st[nt].m = m;
        st[nt].l = l;
#pragma unroll
        for (int jj = 0; jj < J; ++jj) st[nt].o[jj] = o[jj];
    }
    return true;
}

}  // namespace apar
