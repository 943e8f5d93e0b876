// Attention shaped for the matrix cores (16-bit pools): 32x32 products, 128 query rows per workgroup.
//
// Two kernels share one walk:
//   * prefill_bf16: a workgroup takes up to 128 query rows of ONE thread - consecutive query tokens x the
//     q heads of one kv group - and walks that thread's root path under the causal paragraph-tree mask;
//   * attention_units_bf16: a workgroup takes up to 128 query rows of threads that all hold one shared
//     segment (a decode step's stand-alone unit with many rows) and walks a chunk of that segment's
//     blocks; every row sees every filled slot, and the rows' softmax states go out as partial results.
//
// The walk goes in super-blocks of 32 token slots (two KV blocks).  Every wavefront owns 32 rows as the
// N side of 32x32 products:
//
//   S^T[token][row] = K[token][:] . Q[row][:]            8 x mfma_f32_32x32x16_bf16 per super-block
//   O^T[dim][row]  += V^T[dim][token] . P^T[token][row]   8 x mfma_f32_32x32x16_bf16 per super-block
//
// so a lane holds 16 logits per super-block and the per-tile bookkeeping of the online softmax (row
// maximum, the branch that moves the reference, sums) is spread over four times as many elements as in
// the row-tile kernel, and both products run at the full matrix rate.  The accumulator layout of S^T
// (lane = 32 h + n holds tokens 8 j + 4 h + i of row n) is the B-operand layout of P^T once the token
// index of the second product is permuted the same way, so probabilities never move between lanes.
//
// The four wavefronts share the path through LDS in groups of two super-blocks (four KV blocks, double
// buffered, one barrier per group): each wavefront has one block of the next group on its way to LDS, without
// registers in between, while a group is consumed.  Blocks lie in LDS in operand order, as sealed blocks do in
// HBM; a still open one (only the last block of a walk can be) is put into that order once it has landed, and the
// codes of a full fp8 block are widened on their way.
//
// What bounds it: a super-block is 512 cycles of products and some 450 of vector instructions (16 exp2 are 256 of
// them) on the same SIMD, and with one phase after the other a wavefront pair needs 1250 cycles per super-block.  So a
// wavefront's own vector work is issued between its products: the probabilities of one super-block between the K.Q^T
// products of the next one, the maximum over those between the V^T.P^T products, and LDS operands are read beside
// either, into registers that have just become free (218 registers, two wavefronts per SIMD).  Six prompts of 1 k to 8 k
// tokens, 8 kv heads of 4 (1.75 TFLOP): 1.90 -> 1.64 ms, matrix pipe busy 57 % of the time instead of 41 % at a clock that
// falls from 1.94 to 1.79 GHz; own segments of 982 threads, 32 heads, walks of 529: 1.80 -> 1.65 ms.  The direct loads alone,
// phases one after the other as before, take half of that.
// Masks only matter at the end of a row's range: a super-block wholly below a wavefront's first limit is applied
// without masks, one wholly above its last limit is skipped.
#include <hip/hip_runtime.h>

#include <type_traits>

#include "apar_internal.hpp"

namespace apar {

namespace {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __attribute__((__vector_size__(16 * sizeof(float)))) float f32x16;
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));

union Op {  // 16 bytes: a load, or an 8-wide bf16 operand
    u32x4 u;
    bf16x8 b8;
};

constexpr float kSlack = 8.0f;      // a probability may exceed 1 by at most 2^kSlack before the reference moves
constexpr int kTileBytes = 8192;    // one (block, kv head): 4 KiB of K, 4 KiB of V
constexpr int kHalf = 4096;
constexpr int kBufBytes = 4 * kTileBytes;  // one staged group: four blocks, each K half then V half

__device__ __forceinline__ uint32_t pack_pair(float lo, float hi) {  // round to nearest even
    const f32x2 x = {lo, hi};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(x, bf16x2));
}

__device__ __forceinline__ float other_half(float x) {  // the value of lane ^ 32
    const u32x2 r = __builtin_amdgcn_permlane32_swap(__builtin_bit_cast(uint32_t, x), __builtin_bit_cast(uint32_t, x), false, false);
    return __builtin_bit_cast(float, (threadIdx.x & 32) ? r.x : r.y);
}

// fp8 codes in x[0], x[1] times the half's power-of-two scale -> the half's four bf16 pieces x[0..3].
__device__ __forceinline__ void widen(u32x4 (&x)[4], float scale) {
    const u32x4 raw[2] = {x[0], x[1]};
#pragma unroll
    for (int rp = 0; rp < 2; ++rp)
#pragma unroll
        for (int w = 0; w < 4; ++w) {
            x[2 * rp + (w >> 1)][2 * (w & 1)] = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(raw[rp][w], scale, false));
            x[2 * rp + (w >> 1)][2 * (w & 1) + 1] = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(raw[rp][w], scale, true));
        }
}

// What a wavefront brings to the walk.  `len` token slots are filled along the walk's block list
// (entry i of the list is table[i * table_stride]); the lane's row sees slots 0 .. pos.
struct Walk {
    const char* head_base;   // the pool at this kv head
    int64_t block_stride;
    const int32_t* table;
    int table_stride;
    int n_blk;               // blocks that hold a slot some row of the workgroup sees
    int len;
    bool wave_ok;            // the wavefront has rows at all
    int w_first, w_last;     // smallest and largest pos over the wavefront's rows (wavefront-uniform)
    bool row_ok;
    int pos;
    const uint16_t* q_row;   // the lane's query row (any valid row if !row_ok)
    float scale_log2e;
};

// Memory to LDS without a register in between: the lane's 16 bytes at from + ofs go to LDS address lds + 16 lane; dma_half
// brings the three KiB after that too.  Statements of their own rather than the builtin: the compiler takes that one for an
// access that either counter may count, and then has every operand read from LDS wait for all others.  Whoever requests
// waits for vmcnt(0) before anybody reads.  (The wait states cover a scalar register that a vector instruction has just
// written.)
__device__ __forceinline__ void dma_piece(const char* from, uint32_t ofs, uint32_t lds) {
    asm volatile(
        "s_mov_b32 m0, %0\n\t"
        "s_nop 4\n\t"
        "global_load_lds_dwordx4 %1, %2"
        :
        : "s"(lds), "v"(ofs), "s"(from)
        : "memory", "m0");
}
__device__ __forceinline__ void dma_half(const char* from, uint32_t ofs, uint32_t lds) {
    asm volatile(
        "s_mov_b32 m0, %0\n\t"
        "s_nop 4\n\t"
        "global_load_lds_dwordx4 %1, %2\n\t"
        "global_load_lds_dwordx4 %1, %2 offset:1024\n\t"
        "global_load_lds_dwordx4 %1, %2 offset:2048\n\t"
        "global_load_lds_dwordx4 %1, %2 offset:3072"
        :
        : "s"(lds), "v"(ofs), "s"(from)
        : "memory", "m0");
}

// Runs the walk; leaves the lane's share of O^T (dims 32 jj + 16 (j % 2) + 8 (j / 2) + 4 h + i of row n in
// o[jj][4 j + i]), the row's reference m and this lane's half of the row's sum l.
// F8: full blocks hold fp8 codes and two scales; they are widened when they are staged, so that LDS holds the bf16 tile.
template <bool F8>
__device__ __forceinline__ void walk_blocks(const Walk& wk, char* lds, f32x16 (&o)[4], float& m, float& l) {
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int n = lane & 31, h = lane >> 5;   // column (query row) and half of the 32x32 products
    // For the paths that only open blocks take: what is derived from it is not kept in registers over the walk.
    auto recomputed_lane = [&]() {
        int x = lane;
        asm volatile("" : "+v"(x));
        return x;
    };
    const char* head_base = wk.head_base;
    const int64_t block_stride = wk.block_stride;
    const int w_first = wk.w_first, pos = wk.pos;
    const float scale_log2e = wk.scale_log2e;

    // Q as the B operand: lane (n, h) holds dims 8 (2 s + h) .. + 8 of its row for product step s
    Op qv[8];
    {
        const u32x4* qp = reinterpret_cast<const u32x4*>(wk.q_row);
#pragma unroll
        for (int s = 0; s < 8; ++s) qv[s].u = wk.row_ok ? qp[2 * s + h] : u32x4{0u, 0u, 0u, 0u};
    }
#pragma unroll
    for (int jj = 0; jj < 4; ++jj)
#pragma unroll
        for (int i = 0; i < 16; ++i) o[jj][i] = 0.0f;
    m = -INFINITY, l = 0.0f;
    float bias = -INFINITY;  // -m, or -inf as long as the row has seen nothing

    // groups of four blocks (64 token slots)
    const int n_blk = wk.n_blk;
    const int n_grp = (n_blk + 3) / 4;
    const int n_sb = wk.wave_ok ? (wk.w_last >> 5) + 1 : 0;  // super-blocks that some row of the wavefront sees
    // This wavefront stages block `wave` of every group (a group's last blocks may lie past the walk's last block: they
    // are masked, re-read the last one): request() when the group before is about to be consumed, land() when it has been.
    // Sealed blocks lie in LDS as they lie in HBM, and so do open ones once they have landed.
    const uint32_t lds_addr = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)lds;
    u32x4 sk[2], sv[2];        // fp8 pools: the codes of a full block in flight,
    f32x2 ssc = {1.0f, 1.0f};  // and its scales
    auto request = [&](int g) {
        const int blk = min(4 * g + wave, n_blk - 1);
        const int fill = min(16, wk.len - blk * 16);
        const char* tile = head_base + __builtin_amdgcn_readfirstlane(wk.table[blk * wk.table_stride]) * block_stride;
        const uint32_t to = lds_addr + (g & 1) * kBufBytes + wave * kTileBytes;
        if (F8 && fill == 16) {
#pragma unroll
            for (int r = 0; r < 2; ++r) {
                sk[r] = *reinterpret_cast<const u32x4*>(tile + r * 1024 + lane * 16);
                sv[r] = *reinterpret_cast<const u32x4*>(tile + kFp8HalfBytes + r * 1024 + lane * 16);
            }
            ssc = *reinterpret_cast<const f32x2*>(tile + kFp8ScaleOfs);
        } else if (fill == 16) {
            dma_half(tile, lane * 16, to);
            dma_half(tile + kHalf, lane * 16, to + kHalf);
        } else {
            // the walk's last block is still open: row-major.  Piece r of this lane belongs to token row
            // 4r + g4; rows past the fill count re-read row 0 (finite values under probability 0)
            const int ln = recomputed_lane();
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int trow = 4 * r + (ln >> 4) < fill ? 4 * r + (ln >> 4) : 0;
                dma_piece(tile, trow * 256 + (ln & 15) * 16, to + r * 1024);
                dma_piece(tile + kHalf, trow * 256 + (ln & 15) * 16, to + kHalf + r * 1024);
            }
        }
    };
    // (the caller has waited for this wavefront's requests)
    auto land = [&](int g) {
        const int blk = min(4 * g + wave, n_blk - 1);
        const bool sealed = wk.len - blk * 16 >= 16;
        char* dst = lds + (g & 1) * kBufBytes + wave * kTileBytes;
        if (F8 && sealed) {
            // two 16-byte loads hold a half's four pieces at one byte per element (a code times a power of two: exact)
            u32x4 x[4] = {sk[0], sk[1], sk[0], sk[1]};
            widen(x, ssc[0]);
#pragma unroll
            for (int r = 0; r < 4; ++r) *reinterpret_cast<u32x4*>(dst + r * 1024 + lane * 16) = x[r];
            x[0] = sv[0], x[1] = sv[1];
            widen(x, ssc[1]);
#pragma unroll
            for (int r = 0; r < 4; ++r) *reinterpret_cast<u32x4*>(dst + kHalf + r * 1024 + lane * 16) = x[r];
        } else if (!sealed) {
            // piece r of this lane = slot 4r + g4, dims 8c .. 8c + 7 of the open block: put where a sealed one has them
            const int ln = recomputed_lane();
            u32x4 x[4];
#pragma unroll
            for (int r = 0; r < 4; ++r) x[r] = *reinterpret_cast<const u32x4*>(dst + r * 1024 + ln * 16);
            asm volatile("" ::: "memory");  // (lanes read and write each other's pieces)
#pragma unroll
            for (int r = 0; r < 4; ++r) *reinterpret_cast<u32x4*>(dst + bf16_k_offset(4 * r + (ln >> 4), 8 * (ln & 15))) = x[r];
            dst += kHalf;
#pragma unroll
            for (int r = 0; r < 4; ++r) x[r] = *reinterpret_cast<const u32x4*>(dst + r * 1024 + ln * 16);
            asm volatile("" ::: "memory");  // (lanes read and write each other's pieces)
            // V: lanes c, 16 + c, 32 + c, 48 + c hold four slots of the same eight dims and swap words until each has all four
            // slots of two dims (thirty-two 2-byte stores per lane otherwise, eight lanes of each into the same bank)
            const int g4 = ln >> 4, c = ln & 15;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const u32x2 a = __builtin_amdgcn_permlane32_swap(x[r][0], x[r][2], false, false);
                const u32x2 b = __builtin_amdgcn_permlane32_swap(x[r][1], x[r][3], false, false);
                const u32x2 t01 = __builtin_amdgcn_permlane16_swap(a.x, b.x, false, false);  // word g4 of slots 4r, 4r + 1
                const u32x2 t23 = __builtin_amdgcn_permlane16_swap(a.y, b.y, false, false);  // ... 4r + 2, 4r + 3
                const u32x2 even = {(t01.x & 0xffffu) | (t01.y << 16), (t23.x & 0xffffu) | (t23.y << 16)};
                const u32x2 odd = {(t01.x >> 16) | (t01.y & 0xffff0000u), (t23.x >> 16) | (t23.y & 0xffff0000u)};
                *reinterpret_cast<u32x2*>(dst + bf16_v_offset(4 * r, 8 * c + 2 * g4)) = even;
                *reinterpret_cast<u32x2*>(dst + bf16_v_offset(4 * r, 8 * c + 2 * g4 + 1)) = odd;
            }
        }
    };
    // every wavefront's requests have landed, and everyone has read what it needs of the group before
    auto hand_over = [&](int g) {
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_waitcnt(0x0070);  // vmcnt(0) lgkmcnt(0)
        land(g);
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_waitcnt(0xc07f);  // lgkmcnt(0)
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
    };

    // Operands of the super-block whose two blocks lie at `at`.  K: lane (n as token slot, h) reads dims 8 (2 s + h) .. + 8 of
    // slot n % 16 of block n / 16.  V: lane (n as matrix row, h) reads slots 4h .. 4h + 3, then 8 + 4h .. 8 + 4h + 3, of one
    // dim; which of the 32 dims a matrix row stands for is chosen so that eight chunks of 16 bytes - two dims each -
    // serve sixteen lanes (the sixteen lanes of dims c = 0..15 instead would meet in half the banks, twice).
    const int k_lane = (n >> 4) * kTileBytes + (n & 15) * 16 + h * 1024;
    const int v_lane = kHalf + (h * 16 + (n & 7) + 8 * (n >> 4)) * 16 + 8 * ((n >> 3) & 1);
    Op ka[8], va[8];
    float top = -INFINITY;  // the largest of the lane's logits of the super-block to come, unscaled
    auto load_k = [&](const char* at, int k) {
        ka[k].u = *reinterpret_cast<const u32x4*>(at + k_lane + (k & 1) * 2048 + (k >> 1) * 256);
    };
    auto load_v = [&](const char* at, int k) {  // k = 4 block + jj
        const char* p = at + v_lane + (k >> 2) * kTileBytes + (k & 3) * 1024;
        const u32x2 lo = *reinterpret_cast<const u32x2*>(p), hi = *reinterpret_cast<const u32x2*>(p + 512);
        va[k].u = u32x4{lo.x, lo.y, hi.x, hi.y};
    };
    // slot t0 + 8 (i / 4) + 4 h + i % 4 is visible up to the row's pos; only super-blocks near the rows' limits need it
    auto mask = [&](f32x16& s, int t0) {
        if (t0 + 31 > w_first) {
            const int room = pos - t0 - 4 * h;  // visible iff 8 (i / 4) + i % 4 <= room
#pragma unroll
            for (int i = 0; i < 16; ++i) s[i] = (8 * (i >> 2) + (i & 3) <= room) ? s[i] : -INFINITY;
        }
    };
    // If some row ran away from its reference (always so on a row's first super-block): move every row's reference to its
    // running maximum (the two lanes of a row agree on it) and rescale.
    auto settle = [&]() {
        const float t = top * scale_log2e;
        if (__builtin_amdgcn_ballot_w64(t > m + kSlack) != 0) {
            const float mx = fmaxf(t, other_half(t));
            const float m_new = fmaxf(m, mx);
            const float alpha = (m_new == -INFINITY) ? 1.0f : __builtin_amdgcn_exp2f(m - m_new);
            l *= alpha;
#pragma unroll
            for (int jj = 0; jj < 4; ++jj)
#pragma unroll
                for (int i = 0; i < 16; ++i) o[jj][i] *= alpha;
            m = m_new;
            bias = m != -INFINITY ? -m : -INFINITY;
        }
    };
    // Probabilities of the super-block whose logits are s, among the K.Q^T products of the one after it (logits sn, first
    // slot t0n), then the V^T.P^T products among the maximum over sn.  The order is fixed: a wavefront's vector instructions
    // run beside its own products only if they are issued between them.  (After a wavefront's last super-block sn comes from
    // whatever is staged and nobody looks at it: eight products too many per walk, between vector instructions.)
    auto weigh = [&](const f32x16& s, f32x16& sn, int t0n, auto beside_k, auto beside_v) {
        Op pb[2];
        float x0 = __builtin_fmaf(s[0], scale_log2e, bias), x1 = __builtin_fmaf(s[1], scale_log2e, bias);
        float sum0 = 0.0f, sum1 = 0.0f, p0 = 0.0f, p1 = 0.0f;
#pragma unroll
        for (int i = 0; i < 16; ++i) sn[i] = 0.0f;
#pragma unroll
        for (int step = 0; step < 8; ++step) {
            sn = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ka[step].b8, qv[step].b8, sn, 0, 0, 0);
            beside_k(step);
            const float e0 = __builtin_amdgcn_exp2f(x0), e1 = __builtin_amdgcn_exp2f(x1);
            if (step < 7) {
                x0 = __builtin_fmaf(s[2 * step + 2], scale_log2e, bias);
                x1 = __builtin_fmaf(s[2 * step + 3], scale_log2e, bias);
            }
            if (step > 0) {
                sum0 += p0;
                sum1 += p1;
                uint32_t w = pack_pair(p0, p1);
                asm volatile("" : "+v"(w), "+v"(sum0), "+v"(sum1));  // (else they sink below the branch that masks sn)
                pb[(step - 1) >> 2].u[(step - 1) & 3] = w;
            }
            p0 = e0, p1 = e1;
            asm volatile("" : "+v"(p0), "+v"(p1));
            __builtin_amdgcn_sched_barrier(0);
        }
        l += (sum0 + p0) + (sum1 + p1);
        pb[1].u[3] = pack_pair(p0, p1);
        mask(sn, t0n);
        top = fmaxf(sn[0], sn[1]);
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            o[k & 3] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(va[k].b8, pb[k >> 2].b8, o[k & 3], 0, 0, 0);
            beside_v(k);
            if (k > 0) top = fmaxf(fmaxf(top, sn[2 * k]), sn[2 * k + 1]);
            asm volatile("" : "+v"(top));
            __builtin_amdgcn_sched_barrier(0);
        }
    };

    request(0);
    hand_over(0);
    if (n_grp > 1) request(1);
    f32x16 s0, s1;
    int g = 0;
    if (n_sb > 0) {
#pragma unroll
        for (int k = 0; k < 8; ++k) load_k(lds, k);
#pragma unroll
        for (int i = 0; i < 16; ++i) s0[i] = 0.0f;
#pragma unroll
        for (int s = 0; s < 8; ++s) s0 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ka[s].b8, qv[s].b8, s0, 0, 0, 0);
        mask(s0, 0);
        top = s0[0];
#pragma unroll
        for (int i = 1; i < 16; ++i) top = fmaxf(top, s0[i]);
#pragma unroll
        for (int k = 0; k < 8; ++k) load_k(lds + 2 * kTileBytes, k);
        // Group by group; at the top of the loop s0 holds the logits of the group's first super-block and ka the K operands
        // of its second one.  Operands are read from LDS beside products, into registers that have just become free.
        for (; 2 * g < n_sb; ++g) {
            const char* buf = lds + (g & 1) * kBufBytes;
            const char* other = lds + ((g + 1) & 1) * kBufBytes;
            settle();
            weigh(s0, s1, 64 * g + 32, [&](int k) { load_v(buf, k); }, [&](int k) { load_v(buf + 2 * kTileBytes, k); });
            if (2 * g + 1 >= n_sb) break;
            if (g + 1 < n_grp) {
                hand_over(g + 1);
                if (g + 2 < n_grp) request(g + 2);
            }
#pragma unroll
            for (int k = 0; k < 8; ++k) load_k(other, k);
            settle();
            weigh(s1, s0, 64 * g + 64, [](int) {}, [&](int k) { load_k(other + 2 * kTileBytes, k); });
        }
    }
    for (; g + 1 < n_grp; ++g) {  // a wavefront without rows, or whose rows end before the walk does, goes on staging
        hand_over(g + 1);
        if (g + 2 < n_grp) request(g + 2);
    }
    __syncthreads();
}

template <bool F8>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2))) void prefill_bf16(
    const char* __restrict__ pool, const uint16_t* __restrict__ q, const PrefillWg* __restrict__ wgs,
    const int32_t* __restrict__ tables, int n_q, int n_kv, int group, float scale_log2e, uint16_t* __restrict__ out) {
    __shared__ __attribute__((aligned(16))) char lds[2 * kBufBytes];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int n = lane & 31, h = lane >> 5;
    const int kvh = blockIdx.x % n_kv;
    const PrefillWg wg = wgs[blockIdx.x / n_kv];

    // this lane's query row: token tq of the workgroup's chunk, q head hg of the kv group
    const int row = wave * 32 + n;
    const int tq = row / group, hg = row - tq * group;
    const int w_tok0 = (wave * 32) / group;
    Walk wk;
    wk.head_base = pool + (int64_t)kvh * kTileBytes;
    wk.block_stride = (int64_t)n_kv * kTileBytes;
    wk.table = tables + wg.table_ofs;
    wk.table_stride = 1;
    wk.n_blk = (wg.p0 + wg.n_tok - 1) / 16 + 1;  // blocks that hold an attended token
    wk.len = wg.len;
    wk.row_ok = tq < wg.n_tok;
    wk.pos = wg.p0 + (wk.row_ok ? tq : 0);  // position of the row's token in the thread
    // first and last query position of the wavefront
    wk.wave_ok = w_tok0 < wg.n_tok;
    wk.w_first = wg.p0 + w_tok0;
    wk.w_last = wg.p0 + min(wg.n_tok - 1, (wave * 32 + 31) / group);
    const int64_t qrow = ((int64_t)(wg.q_row0 + (wk.row_ok ? tq : 0)) * n_q) + kvh * group + hg;
    wk.q_row = q + qrow * 128;
    wk.scale_log2e = scale_log2e;
    f32x16 o[4];
    float m, l;
    walk_blocks<F8>(wk, lds, o, m, l);

    // Normalise and write.  The rows go through LDS (the walk ended with a barrier) so that a store instruction writes
    // four whole rows of 256 bytes: a lane holds its row in runs of four dims, and stores of 8 bytes per lane, 16 per
    // row, leave the L2 as partial lines (80 requests, 480 segments of 107 tokens, walks of 300, 32 heads, 0.85 GB of
    // queries and outputs: 1580 us with non-temporal stores of 8 bytes, 678 with plain ones, 650 this way).
    const float lt = l + other_half(l);
    const float inv = 1.0f / lt;
    constexpr int kStride = 256 + 16;  // padded: the rows of a column of lanes start in different banks
    char* rows = lds + wave * 32 * kStride;
#pragma unroll
    for (int jj = 0; jj < 4; ++jj)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            u32x2 pk;
            pk.x = pack_pair(o[jj][4 * j + 0] * inv, o[jj][4 * j + 1] * inv);
            pk.y = pack_pair(o[jj][4 * j + 2] * inv, o[jj][4 * j + 3] * inv);
            *reinterpret_cast<u32x2*>(rows + n * kStride + (32 * jj + 16 * (j & 1) + 8 * (j >> 1) + 4 * h) * 2) = pk;
        }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll
    for (int it = 0; it < 8; ++it) {
        const int r = 4 * it + (lane >> 4);
        const u32x4 x = *reinterpret_cast<const u32x4*>(rows + r * kStride + (lane & 15) * 16);
        const int t2 = (wave * 32 + r) / group, h2 = wave * 32 + r - t2 * group;
        if (t2 >= wg.n_tok) continue;
        uint16_t* dst = out + (((int64_t)(wg.q_row0 + t2) * n_q) + kvh * group + h2) * 128;
        __builtin_nontemporal_store(x, reinterpret_cast<u32x4*>(dst) + (lane & 15));
    }
}

// Stand-alone units of a decode plan with many rows.  The workgroup descriptor's shared tile list is the
// chunk of the segment (full blocks first, the open one last); its first wavefront entry names the
// threads: depth-first ranks grp_lo / n_slices .. + n_grp / n_slices, rows_per_thread rows each, laid
// flat over the 128 rows; part_base is the first thread's partial-result row for this chunk.
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2))) void attention_units_bf16(
    const char* __restrict__ pool, const uint16_t* __restrict__ q, PlanDev plan, int wg_first, int n_cand, int n_q,
    int n_kv, int group, float scale_log2e, PartialBuf part) {
    __shared__ __attribute__((aligned(16))) char lds[2 * kBufBytes];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int n = lane & 31, h = lane >> 5;
    const int kvh = blockIdx.x % n_kv;
    const WgDesc* wg = plan.wgs + wg_first + blockIdx.x / n_kv;
    const TileRef* tiles = plan.tiles + wg->coop_ofs;
    const int n_blk = wg->n_coop;
    const int rpt = plan.rows_per_thread;
    const int rank0 = wg->w[0].grp_lo / plan.n_slices, n_thr = wg->w[0].n_grp / plan.n_slices;
    const int last_fill = (tiles[n_blk - 1].meta >> 20) & 31;

    const int row = wave * 32 + n;
    const int tr = row / rpt, within = row - tr * rpt;
    Walk wk;
    wk.head_base = pool + (int64_t)kvh * kTileBytes;
    wk.block_stride = (int64_t)n_kv * kTileBytes;
    wk.table = unwritten(&tiles[0].blk);
    wk.table_stride = sizeof(TileRef) / sizeof(int32_t);
    wk.n_blk = n_blk;
    wk.len = (n_blk - 1) * 16 + last_fill;
    wk.row_ok = tr < n_thr;
    wk.pos = wk.len - 1;  // every row sees every filled slot
    wk.wave_ok = wave * 32 < n_thr * rpt;
    wk.w_first = wk.w_last = wk.len - 1;
    const int tr_ok = wk.row_ok ? tr : 0, within_ok = wk.row_ok ? within : 0;
    const int listed = plan.dfs_threads ? plan.dfs_threads[rank0 + tr_ok] : rank0 + tr_ok;
    const int cc = within_ok / group, hq = kvh * group + (within_ok - cc * group);
    wk.q_row = q + (((int64_t)listed * n_cand + cc) * n_q + hq) * 128;
    wk.scale_log2e = scale_log2e;
    f32x16 o[4];
    float m, l;
    walk_blocks<false>(wk, lds, o, m, l);

    // the row's state goes out as a partial result
    const float lt = l + other_half(l);
    if (!wk.row_ok) return;
    const int64_t slot = ((int64_t)(wg->w[0].part_base + tr) * n_cand + cc) * n_q + hq;
    float* dst = part.o + slot * 128 + 4 * h;
    auto write = [&](auto stream) {
#pragma unroll
        for (int jj = 0; jj < 4; ++jj)
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const f32x4 v = {o[jj][4 * j + 0], o[jj][4 * j + 1], o[jj][4 * j + 2], o[jj][4 * j + 3]};
                f32x4* to = reinterpret_cast<f32x4*>(dst + 32 * jj + 16 * (j & 1) + 8 * (j >> 1));
                if constexpr (decltype(stream)::value) __builtin_nontemporal_store(v, to);
                else *to = v;
            }
    };
    if (part.stream) {
        asm volatile("" ::: "memory");  // (before and after: else the two branches' stores become one, without the hint)
        write(std::true_type{});
        asm volatile("" ::: "memory");
    } else {
        write(std::false_type{});
    }
    if (h == 0) {
        part.ml[slot * 2] = m;
        part.ml[slot * 2 + 1] = lt;
    }
}

}  // namespace

hipError_t launch_prefill_bf16(const Shape& s, const void* pool, const void* q, const PrefillWg* wgs,
                               const int32_t* tables, int n_wg, void* out, hipStream_t st) {
    if (n_wg <= 0) return hipSuccess;
    const int64_t grid = (int64_t)n_wg * s.n_kv;
    if (grid > 0x7fffffff) return hipErrorInvalidValue;
    if (s.fp8_sealed)
        hipLaunchKernelGGL(prefill_bf16<true>, dim3((unsigned)grid), dim3(256), 0, st, (const char*)pool, (const uint16_t*)q, wgs,
                           tables, s.n_q, s.n_kv, s.group, s.scale_log2e, (uint16_t*)out);
    else
        hipLaunchKernelGGL(prefill_bf16<false>, dim3((unsigned)grid), dim3(256), 0, st, (const char*)pool, (const uint16_t*)q, wgs,
                           tables, s.n_q, s.n_kv, s.group, s.scale_log2e, (uint16_t*)out);
    return hipGetLastError();
}

hipError_t launch_attention_units_bf16(const Shape& s, const void* pool, const void* q, const PlanDev& plan,
                                       int wg_first, int n_wg, int n_cand, PartialBuf part, hipStream_t st) {
    if (n_wg <= 0) return hipSuccess;
    const int64_t grid = (int64_t)n_wg * s.n_kv;
    if (grid > 0x7fffffff) return hipErrorInvalidValue;
    hipLaunchKernelGGL(attention_units_bf16, dim3((unsigned)grid), dim3(256), 0, st, (const char*)pool,
                       (const uint16_t*)q, plan, wg_first, n_cand, s.n_q, s.n_kv, s.group, s.scale_log2e, part);
    return hipGetLastError();
}

}  // namespace apar
