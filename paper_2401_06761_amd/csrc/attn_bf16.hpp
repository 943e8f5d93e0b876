// What the 16-bit decode kernels are made of (device side): operands, products, online softmax, candidates.
#pragma once

#include <hip/hip_runtime.h>

#include <type_traits>

#include "apar_internal.hpp"
#include "attn_split.hpp"

namespace apar {

namespace {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __attribute__((__vector_size__(4 * sizeof(short)))) short s16x4;
typedef __attribute__((address_space(3))) s16x4 lds_s16x4;
typedef __attribute__((__vector_size__(4 * sizeof(float)))) float f32x4;
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));

union Frag {  // 16 bytes seen as a load, as an 8-wide bf16 operand, or as two 4-wide ones
    u32x4 u;
    bf16x8 b8;
    s16x4 h4[2];
};

constexpr float kSlack = 8.0f;  // a probability may exceed 1 by at most 2^kSlack before the reference moves
constexpr int kTileBytes = 8192;

// The 16 rows of one wavefront: query operands and running softmax state.
struct RowState {
    Frag q[4];
    f32x4 o[8];
    float m, l;
};

// S^T = K.Q^T for one tile: raw dot products, tokens 4*g4 .. 4*g4+3 of this lane's row.
__device__ __forceinline__ f32x4 products(const Frag (&k)[4], const RowState& st) {
    f32x4 s = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) s = __builtin_amdgcn_mfma_f32_16x16x32_bf16(k[kk].b8, st.q[kk].b8, s, 0, 0, 0);
    return s;
}

// Token slots whose bit is clear in tok_mask (per lane, i.e. per query row) get a product of -inf and
// hence probability 0.  Only needed for tiles that are not full and for candidate tiles.
__device__ __forceinline__ void mask_tokens(f32x4& s, uint32_t tok_mask, int g4) {
    const uint32_t mine = tok_mask >> (4 * g4);
#pragma unroll
    for (int i = 0; i < 4; ++i) s[i] = ((mine >> i) & 1u) ? s[i] : -INFINITY;
}

__device__ __forceinline__ uint32_t pack_bf16_pair(float lo, float hi) {  // round to nearest even, one instruction
    const f32x2 x = {lo, hi};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(x, bf16x2));
}

// Two 16-byte pieces of fp8 codes (one half of a sealed fp8 tile as this lane holds it) times the half's
// power-of-two scale -> the four bf16 operand pieces of the half.
__device__ __forceinline__ void fp8_operands(const u32x4 (&raw)[2], float scale, Frag (&f)[4]) {
#pragma unroll
    for (int rp = 0; rp < 2; ++rp)
#pragma unroll
        for (int w = 0; w < 4; ++w) {
            Frag& dst = f[2 * rp + (w >> 1)];
            dst.u[2 * (w & 1)] = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(raw[rp][w], scale, false));
            dst.u[2 * (w & 1) + 1] = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(raw[rp][w], scale, true));
        }
}

// Online softmax step, first half: if some row's logits ran away from its reference (always so for a
// row's first tile, whose reference is still -inf), move every row's reference to its running maximum
// (the four lanes of a row agree on it) and rescale what was summed.  Rare, hence behind a branch.
__device__ __forceinline__ float top_logit(const f32x4& s, bool in_range, float scale_log2e) {
    return in_range ? fmaxf(fmaxf(s[0], s[1]), fmaxf(s[2], s[3])) * scale_log2e : -INFINITY;
}

__device__ __forceinline__ void raise_reference(RowState& st, float top) {
    float mx = fmaxf(top, __shfl_xor(top, 16, 64));
    mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
    const float m_new = fmaxf(st.m, mx);
    // a row that has seen nothing yet keeps m = -inf and sums of zero
    const float alpha = (m_new == -INFINITY) ? 1.0f : __builtin_amdgcn_exp2f(st.m - m_new);
    st.l *= alpha;
#pragma unroll
    for (int j = 0; j < 8; ++j) st.o[j] *= alpha;
    st.m = m_new;
}

__device__ __forceinline__ void move_reference(RowState& st, const f32x4& s, bool in_range, float scale_log2e) {
    const float top = top_logit(s, in_range, scale_log2e);
    if (__builtin_amdgcn_ballot_w64(top > st.m + kSlack) != 0) raise_reference(st, top);
}

// The same for all row tiles of a wavefront behind ONE branch (a branch on a vector compare costs
// the wavefront some eighty cycles): if any row of any tile ran away, every touched tile's rows move
// to their running maxima, which is always allowed.
template <int NT>
__device__ __forceinline__ void move_references(RowState (&st)[NT], const f32x4 (&s)[NT], const bool (&on)[NT],
                                                const bool (&in_range)[NT], float scale_log2e) {
    float top[NT];
    bool ran_away = false;
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
        top[nt] = on[nt] ? top_logit(s[nt], in_range[nt], scale_log2e) : -INFINITY;
        ran_away = ran_away || top[nt] > st[nt].m + kSlack;
    }
    if (__builtin_amdgcn_ballot_w64(ran_away) != 0) {
#pragma unroll
        for (int nt = 0; nt < NT; ++nt)
            if (on[nt]) raise_reference(st[nt], top[nt]);
    }
}

// Second half, straight-line: probabilities and O^T += V^T.P^T for one tile that applies to this lane's
// row iff in_range.  The softmax scale and the reference are folded into one fused multiply-add per
// logit; rows outside the range, and slots masked to -inf, get probability exp2(-inf) = 0.  V rows of
// unfilled slots must be finite (the loaders hand over a copy of row 0 for them): 0 * V is added.
__device__ __forceinline__ void weigh_values(const Frag (&v)[4], RowState& st, const f32x4& s, bool in_range,
                                             float scale_log2e) {
    const float bias = (in_range & (st.m != -INFINITY)) ? -st.m : -INFINITY;
    float p[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) p[i] = __builtin_amdgcn_exp2f(__builtin_fmaf(s[i], scale_log2e, bias));
    st.l += (p[0] + p[1]) + (p[2] + p[3]);
    union {
        uint32_t w[2];
        s16x4 h;
    } pp;
    pp.w[0] = pack_bf16_pair(p[0], p[1]);
    pp.w[1] = pack_bf16_pair(p[2], p[3]);
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        st.o[2 * r] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(v[r].h4[0], pp.h, st.o[2 * r], 0, 0, 0);
        st.o[2 * r + 1] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(v[r].h4[1], pp.h, st.o[2 * r + 1], 0, 0, 0);
    }
}

__device__ __forceinline__ void accumulate(const Frag (&v)[4], RowState& st, const f32x4& s, bool in_range,
                                           float scale_log2e) {
    move_reference(st, s, in_range, scale_log2e);
    weigh_values(v, st, s, in_range, scale_log2e);
}

// V^T operand pieces out of a ROW-MAJOR V half held in LDS (rows `stride` bytes apart):
// piece r holds V[tokens 4g..4g+3][dim 32r + c] and V[tokens 4g..4g+3][dim 32r + 16 + c].  The LDS read that transposes:
// sixteen lanes name the 8-byte pieces of a 4 x 16 corner, four lanes a row, and lane c gets column c.
__device__ __forceinline__ void v_operands_from_rows(const char* vrows, int stride, int g4, int c, Frag (&v)[4]) {
    const char* corner = vrows + (4 * g4 + (c >> 2)) * stride + (c & 3) * 8;
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int hh = 0; hh < 2; ++hh)
            v[r].h4[hh] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(corner + (32 * r + 16 * hh) * 2));
}

constexpr int kOpenRowStride = 272;                 // padded, so the four token groups hit different LDS banks
constexpr int kOpenScratch = 16 * kOpenRowStride;   // one wavefront's row-major V half

// Multi-candidate call: each thread's candidates are one more tile of at most 8 token rows (row-major, a row every n_kv * 128
// elements), visible to a row only where its mask bit is set.  scratch: kOpenScratch bytes of the wavefront's own.
template <int NT>
__device__ __forceinline__ void attend_candidates(RowState (&st)[NT], char* scratch, const PlanDev& plan, const WaveItem& wi,
                                                  const uint16_t* __restrict__ cand_k, const uint16_t* __restrict__ cand_v,
                                                  const uint8_t* __restrict__ cand_mask, const int (&my_j)[NT], int within, int n_cand,
                                                  int n_kv, int kvh, int group, float scale_log2e) {
    const int lane = threadIdx.x & 63, g4 = lane >> 4, c = lane & 15;
    const int n_sl = plan.n_slices, rps = plan.rows_per_slice;
    const int rank_lo = wi.grp_lo / n_sl, rank_hi = (wi.grp_lo + wi.n_grp - 1) / n_sl;
    const int64_t tok_stride = (int64_t)n_kv * 256;  // bytes between candidate rows of one kv head
    for (int ru = rank_lo; ru <= rank_hi; ++ru) {
        const int listed_u = plan.dfs_threads ? plan.dfs_threads[ru] : ru;
        const int64_t base = ((int64_t)listed_u * n_cand * n_kv + kvh) * 256;
        const char* kb = reinterpret_cast<const char*>(cand_k) + base;
        const char* vb = reinterpret_cast<const char*>(cand_v) + base;
        Frag kc[4], vc[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            // rows past the last candidate: re-read candidate 0 (finite values under probability 0)
            kc[r].u = *reinterpret_cast<const u32x4*>(kb + (c < n_cand ? c : 0) * tok_stride + g4 * 64 + r * 16);
            const int row = 4 * r + g4 < n_cand ? 4 * r + g4 : 0;
            const u32x4 vr = *reinterpret_cast<const u32x4*>(vb + row * tok_stride + c * 16);
            *reinterpret_cast<u32x4*>(scratch + (4 * r + g4) * kOpenRowStride + c * 16) = vr;
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        v_operands_from_rows(scratch, kOpenRowStride, g4, c, vc);
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
            uint32_t tm = 0;
            if (my_j[nt] != 0x7fff) {
                const int grp = wi.grp_lo + my_j[nt];
                const int rk = grp / n_sl, r2 = (grp - rk * n_sl) * rps + within;
                if (rk == ru) tm = cand_mask[(int64_t)listed_u * n_cand + r2 / group];
            }
            if (__builtin_amdgcn_ballot_w64(tm != 0) == 0) continue;
            f32x4 sc = products(kc, st[nt]);
            mask_tokens(sc, tm, g4);
            accumulate(vc, st[nt], sc, tm != 0, scale_log2e);
        }
    }
}

// The scale of a full fp8 tile's half, by a scalar load (full blocks are not written while a kernel reads them).
__device__ __forceinline__ float scale_at(const char* p) { return *(const float __attribute__((address_space(4)))*)p; }

constexpr int kSplitState = 8 * 1024 + 512;  // eight accumulator quads, reference and share of the sum per lane

template <bool SPLIT, bool INLINE>
__device__ __forceinline__ Slice unit_of_block(PlanDev& plan, int wg_first, int n_kv) {
    if constexpr (INLINE) plan_from_arguments(plan);
    Slice slice;
    if constexpr (SPLIT) {
        slice = slice_of_block(plan.split, wg_first, n_kv);
    } else {
        slice.wg = wg_first + blockIdx.x / n_kv;
    }
    return slice;
}

}  // namespace

}  // namespace apar
