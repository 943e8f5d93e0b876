// Decode attention over bf16 KV tiles: calls of few units (PlanDev::few; the rule stands in apar_pool.cpp).
//
// Units without shared lists, of one row tile or two.  What bounds such a call is one wavefront's chain of latencies; what it was made
// of by the kernel for any unit (one request of five threads, 32 heads, 26 k cycles): descriptor and queries 3.5 k, a tile 1180 with one
// in flight (products and softmax take 350), an open tile 1600 (its K gathered sixteen bytes a row), fold by one wavefront and output
// 4.5 k.  So here two tiles (three of fp8 codes) are on their way at any time, open tiles among them: every tile is fetched the same
// way, KiB by KiB, and an open one's rows are put into operand order through LDS.  The four wavefronts of a divided list fold and write
// a quarter of the dims each.  13.5 -> 8.6 us per call (8.9 before their tables were packed); with 8 kv heads 14.4 -> 8.5 (in two units instead of one of two wavefronts).
// One compute unit takes 50 bytes per cycle however many loads are on their way, 640 cycles per tile and wavefront, so that a tile
// takes 720 with two on their way.  Two row tiles (where units of 16 rows would read shared segments too often): the queries lie in
// LDS, which leaves registers for the two tiles (202; four requests of 4 k tokens, group 8 32.2 -> 27.8 us).
#include <hip/hip_runtime.h>

#include <cstring>
#include <type_traits>

#include "attn_bf16.hpp"

namespace apar {

namespace {

template <int NT>
struct FewLds {
    // one row tile: the states lie apart from the scratch, and nobody waits before leaving one; two: queries behind the scratch, the
    // states, row tile by row tile, where both were
    static constexpr int kQueries = 4 * kOpenScratch;
    static constexpr int kStates = NT == 1 ? 4 * kOpenScratch : 0;
    static constexpr int kBytes = NT == 1 ? kStates + 4 * kSplitState : kQueries + 4 * NT * 4096;
    static_assert(NT == 1 || kBytes >= 4 * kSplitState, "states of one row tile");
};

template <int NT>
struct FewWalk {
    const char* head_base;
    int64_t block_stride;
    float scale_log2e;
    int my_j[NT];     // row group of this lane's row of each row tile, or 0x7fff
    int cap;          // row groups per row tile
    char* scratch;    // kOpenScratch bytes of LDS
    const char* q;    // NT = 2: the lane's query pieces in LDS, 1 KiB apart, row tile after row tile (NT = 1: in registers)
    int lane;

    __device__ __forceinline__ void queries(RowState& st, int nt) const {
        if constexpr (NT > 1) {
            asm volatile("" ::: "memory");  // (read for every tile, not kept)
#pragma unroll
            for (int kk = 0; kk < 4; ++kk) st.q[kk].u = *reinterpret_cast<const u32x4*>(q + (nt * 4 + kk) * 1024);
        }
    }
};

// A tile on its way: its rows or operand pieces (CODES: the codes of a full fp8 tile).
template <bool CODES, int NT>
struct FewTile {
    Frag k[4], v[4];
    u32x4 k8[CODES ? 2 : 1], v8[CODES ? 2 : 1];
    float ks, vs;
    int meta;

    __device__ __forceinline__ void fetch_k(const FewWalk<NT>& w, const char* tile, int rows) {
        if constexpr (CODES) {
#pragma unroll
            for (int r = 0; r < 2; ++r) k8[r] = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(tile + w.lane * 16 + r * 1024));
            ks = scale_at(tile + kFp8ScaleOfs);
        } else {
            fetch_half(w, tile, rows, k);
        }
    }
    __device__ __forceinline__ void fetch_v(const FewWalk<NT>& w, const char* tile, int rows) {
        if constexpr (CODES) {
#pragma unroll
            for (int r = 0; r < 2; ++r)
                v8[r] = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(tile + kFp8HalfBytes + w.lane * 16 + r * 1024));
            vs = scale_at(tile + kFp8ScaleOfs + 4);
        } else {
            fetch_half(w, tile + 4096, rows, v);
        }
    }
    // The half's KiB r: the operands' piece r of a full tile, token rows 4r .. 4r + 3 of an open one (rows that are not filled: row 0).
    __device__ __forceinline__ static void fetch_half(const FewWalk<NT>& w, const char* half, int rows, Frag (&f)[4]) {
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const uint32_t at = 4 * r + (w.lane >> 4) < rows ? r * 1024 + w.lane * 16 : (w.lane & 15) * 16;
            f[r].u = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(half + at));
        }
    }
    __device__ __forceinline__ static void rows_to_lds(const FewWalk<NT>& w, const Frag (&f)[4]) {
#pragma unroll
        for (int r = 0; r < 4; ++r) *reinterpret_cast<u32x4*>(w.scratch + (4 * r + (w.lane >> 4)) * kOpenRowStride + (w.lane & 15) * 16) = f[r].u;
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    }
    // Takes the tile; meanwhile the next one for these registers, `rows` rows of it, is fetched (rows = 1: there is none, and a row of
    // the list's last tile comes instead, so that no load lies behind a branch).
    template <bool MORE>
    __device__ __forceinline__ void take(const FewWalk<NT>& w, RowState (&st)[NT], const char* next, int next_meta, int rows) {
        const int g4 = w.lane >> 4, c = w.lane & 15;
        const int lo = meta & 1023, hi = (meta >> 10) & 1023, valid = (meta >> 20) & 31;
        const bool causal = meta >> 30, open = !CODES && valid < kBlockTokens;
        bool on[NT], in_range[NT];
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
            on[nt] = NT == 1 || (lo < (nt + 1) * w.cap && hi > nt * w.cap);  // (wavefront-uniform)
            in_range[nt] = w.my_j[nt] >= lo && w.my_j[nt] < hi;
        }
        if constexpr (CODES) {
            fp8_operands(k8, ks, k);
        } else if (open) {
            rows_to_lds(w, k);
#pragma unroll
            for (int r = 0; r < 4; ++r) k[r].u = *reinterpret_cast<const u32x4*>(w.scratch + c * kOpenRowStride + g4 * 64 + r * 16);
            __builtin_amdgcn_wave_barrier();
        }
        f32x4 s[NT];
#pragma unroll
        for (int nt = 0; nt < NT; ++nt)
            if (on[nt]) {
                w.queries(st[nt], nt);
                s[nt] = products(k, st[nt]);
            }
        if constexpr (MORE) fetch_k(w, next, rows);
        if (open || causal) {
            const int first = (meta >> 25) & 31;
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) {
                const int limit = causal ? min(valid, max(0, first + w.my_j[nt] - lo)) : valid;
                if (on[nt]) mask_tokens(s[nt], (1u << limit) - 1u, g4);
            }
        }
        move_references<NT>(st, s, on, in_range, w.scale_log2e);
        if constexpr (CODES) {
            fp8_operands(v8, vs, v);
        } else if (open) {
            rows_to_lds(w, v);
            v_operands_from_rows(w.scratch, kOpenRowStride, g4, c, v);
            __builtin_amdgcn_wave_barrier();
        }
#pragma unroll
        for (int nt = 0; nt < NT; ++nt)
            if (on[nt]) weigh_values(v, st[nt], s[nt], in_range[nt], w.scale_log2e);
        if constexpr (MORE) fetch_v(w, next, rows);
        meta = next_meta;
    }
};

// A list of tiles; PACKED: as pack_few_tile leaves them.
template <bool PACKED>
struct FewRefs {
    const TileRef* p;
    __device__ __forceinline__ TileRef operator[](int i) const {
        if constexpr (PACKED) return unpack_few_tile(reinterpret_cast<const uint32_t*>(p)[i]);
        else return p[i];
    }
    __device__ __forceinline__ FewRefs from(int i) const {
        if constexpr (PACKED) return {reinterpret_cast<const TileRef*>(reinterpret_cast<const uint32_t*>(p) + i)};
        else return {p + i};
    }
};

template <bool CODES, int NT, bool PACKED>
struct FewList {
    static constexpr int kSets = CODES ? 3 : 2;
    FewTile<CODES, NT> set[kSets];
    FewRefs<PACKED> list;
    int n;

    __device__ __forceinline__ void start(const FewWalk<NT>& w) {
        if (n <= 0) return;
        TileRef ref[kSets];
#pragma unroll
        for (int i = 0; i < kSets; ++i) ref[i] = list[min(i, n - 1)];
#pragma unroll
        for (int i = 0; i < kSets; ++i) {
            const char* tile = w.head_base + ref[i].blk * w.block_stride;
            const int rows = i < n ? (ref[i].meta >> 20) & 31 : 1;
            set[i].meta = ref[i].meta;
            __builtin_amdgcn_sched_barrier(0);  // in this order, which the loop keeps
            set[i].fetch_k(w, tile, rows);
            __builtin_amdgcn_sched_barrier(0);
            set[i].fetch_v(w, tile, rows);
            __builtin_amdgcn_sched_barrier(0);
        }
    }
    __device__ __forceinline__ void walk(const FewWalk<NT>& w, RowState (&st)[NT]) {
        if (n <= 0) return;
        int t = 0;
        for (; t + kSets <= n; t += kSets) {
#pragma unroll
            for (int i = 0; i < kSets; ++i) {
                const TileRef ref = list[min(t + kSets + i, n - 1)];
                set[i].template take<true>(w, st, w.head_base + ref.blk * w.block_stride, ref.meta, t + kSets + i < n ? (ref.meta >> 20) & 31 : 1);
            }
        }
#pragma unroll
        for (int i = 0; i + 1 < kSets; ++i)
            if (t + i < n) set[i].template take<false>(w, st, nullptr, 0, 0);
    }
};

template <int NT, bool F8, bool SPLIT, bool PACKED>
__device__ __forceinline__ void attend_few(char* lds, const Slice& slice, const char* __restrict__ pool, const uint16_t* __restrict__ q,
                                           const PlanDev& plan, int n_cand, int n_q, int n_kv, int group, float scale_log2e,
                                           const PartialBuf& part, const uint16_t* __restrict__ cand_k, const uint16_t* __restrict__ cand_v,
                                           const uint8_t* __restrict__ cand_mask, uint16_t* __restrict__ out) {
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int g4 = lane >> 4, c = lane & 15;
    const int kvh = blockIdx.x % n_kv;
    WaveItem wi;
    int own_full;
    if constexpr (PACKED) {
        const uint32_t* w = reinterpret_cast<const uint32_t*>(plan.wgs) + (slice.wg * 4 + wave) * kFewWaveWords;
        wi = unpack_few_wave(w[0], w[1], own_full);
    } else {
        const WgDesc* wg = plan.wgs + slice.wg;
        wi = wg->w[wave];
        own_full = min(wg->n_full[wave], wi.n_tiles);
    }
    if constexpr (SPLIT) cut_list(slice, wi.tile_ofs, wi.n_tiles, own_full);
    if (wi.n_grp == 0) return;  // (never one of the four wavefronts of a divided list)
    const FewRefs<PACKED> mine = FewRefs<PACKED>{plan.tiles}.from(wi.tile_ofs);

    // column c of row tile nt is row `within` of the wavefront's row group nt * cap + c / rps
    const int rps = plan.rows_per_slice, n_sl = plan.n_slices, cap = 16 / rps;
    const int jc = c / rps, within = c - jc * rps;
    char* scratch = lds + wave * kOpenScratch;
    char* my_q = lds + FewLds<NT>::kQueries + wave * NT * 4096 + lane * 16;
    FewWalk<NT> walk{pool + (int64_t)kvh * kTileBytes, (int64_t)n_kv * kTileBytes, scale_log2e, {}, cap, scratch, my_q, lane};
    RowState st[NT];
    int64_t qrow[NT];  // -1: no row
    int64_t slot[NT];  // of the row's partial result
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
        const int j = nt * cap + jc, grp = wi.grp_lo + j, rank = grp / n_sl, rr = (grp - rank * n_sl) * rps + within;
        const bool ok = jc < cap && j < wi.n_grp && rr < plan.rows_per_thread;
        const int listed = ok ? (plan.dfs_threads ? plan.dfs_threads[rank] : rank) : 0;
        const int cc = ok ? rr / group : 0, hq = kvh * group + (ok ? rr - cc * group : 0);
        const int64_t row = ((int64_t)listed * n_cand + cc) * n_q + hq;
        walk.my_j[nt] = ok ? j : 0x7fff;
        qrow[nt] = ok ? row : -1;
        slot[nt] = ((int64_t)(wi.part_base + rank - wi.grp_lo / n_sl) * n_cand + cc) * n_q + hq;
        st[nt].m = -INFINITY;
        st[nt].l = 0.0f;
#pragma unroll
        for (int jj = 0; jj < 8; ++jj) st[nt].o[jj] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
        const u32x4* qp = reinterpret_cast<const u32x4*>(q + row * 128 + g4 * 32);
#pragma unroll
        for (int kk = 0; kk < 4; ++kk) {  // (a column without a row: some row's queries, for no tile)
            if constexpr (NT == 1) st[nt].q[kk].u = qp[kk];
            else *reinterpret_cast<u32x4*>(my_q + (nt * 4 + kk) * 1024) = qp[kk];
        }
    }
    if constexpr (F8) {  // full tiles are codes, open ones rows
        FewList<true, NT, PACKED> codes;
        FewList<false, NT, PACKED> rows;
        codes.list = mine, codes.n = own_full;
        rows.list = mine.from(own_full), rows.n = wi.n_tiles - own_full;
        codes.start(walk);
        if constexpr (NT == 1) rows.start(walk);
        codes.walk(walk, st);
        if constexpr (NT > 1) rows.start(walk);
        rows.walk(walk, st);
    } else {
        FewList<false, NT, PACKED> tiles;
        tiles.list = mine, tiles.n = wi.n_tiles;
        tiles.start(walk);
        tiles.walk(walk, st);
    }
    const bool divided = wi.flags & kWaveSplit;
    if ((wi.flags & kWaveDirect) && cand_mask != nullptr && (!SPLIT || slice.s == 0) && (!divided || wave == 0)) {
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) walk.queries(st[nt], nt);
        attend_candidates<NT>(st, scratch, plan, wi, cand_k, cand_v, cand_mask, walk.my_j, within, n_cand, n_kv, kvh, group, scale_log2e);
    }

    auto write = [&](auto quads, int j0, int nt) {  // quads j0 .. of the lane's row of row tile nt
        constexpr int J = decltype(quads)::value;
        float l = st[nt].l;
        l += __shfl_xor(l, 16, 64);
        l += __shfl_xor(l, 32, 64);
        if (qrow[nt] < 0) return;
        if (wi.flags & kWaveDirect) {
            const float inv = 1.0f / l;
            uint16_t* dst = out + qrow[nt] * 128 + 4 * g4;
#pragma unroll
            for (int jj = 0; jj < J; ++jj) {
                u32x2 pk;
                pk.x = pack_bf16_pair(st[nt].o[jj][0] * inv, st[nt].o[jj][1] * inv);
                pk.y = pack_bf16_pair(st[nt].o[jj][2] * inv, st[nt].o[jj][3] * inv);
                *reinterpret_cast<u32x2*>(dst + 16 * (j0 + jj)) = pk;
            }
        } else {
#pragma unroll
            for (int jj = 0; jj < J; ++jj) *reinterpret_cast<f32x4*>(part.o + slot[nt] * 128 + 4 * g4 + 16 * (j0 + jj)) = st[nt].o[jj];
            if (g4 == 0 && j0 == 0) {
                part.ml[slot[nt] * 2] = st[nt].m;
                part.ml[slot[nt] * 2 + 1] = l;
            }
        }
    };
    if (!divided) {
        if constexpr (SPLIT)
            if (!fold_slices<NT, 8>(plan.split, slice, n_kv, kvh, wave, 4, lane, st)) return;
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) write(std::integral_constant<int, 8>{}, 0, nt);
        return;
    }
    // the four wavefronts hold the same rows over different tiles: every one folds two of the eight accumulator quads
    // (not __syncthreads: it would wait for the rows fetched past the lists' ends)
    auto meet = [] {
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_waitcnt(0xc07f);  // lgkmcnt(0)
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
    };
    char* states = lds + FewLds<NT>::kStates;
    const int j0 = 2 * wave;
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
        if (NT > 1) meet();  // (everyone is done with what the states overlap)
        {
            char* to = states + wave * kSplitState;
#pragma unroll
            for (int jj = 0; jj < 8; ++jj) *reinterpret_cast<f32x4*>(to + (jj * 64 + lane) * 16) = st[nt].o[jj];
            *reinterpret_cast<f32x2*>(to + 8 * 1024 + lane * 8) = f32x2{st[nt].m, st[nt].l};
        }
        meet();
        f32x2 ml[4];
        f32x4 o[4][2];
#pragma unroll
        for (int w2 = 0; w2 < 4; ++w2) {
            const char* from = states + w2 * kSplitState;
            ml[w2] = *reinterpret_cast<const f32x2*>(from + 8 * 1024 + lane * 8);
#pragma unroll
            for (int jj = 0; jj < 2; ++jj) o[w2][jj] = *reinterpret_cast<const f32x4*>(from + ((j0 + jj) * 64 + lane) * 16);
        }
        const float mx = fmaxf(fmaxf(ml[0].x, ml[1].x), fmaxf(ml[2].x, ml[3].x));
        st[nt].m = mx;
        st[nt].l = 0.0f;
#pragma unroll
        for (int jj = 0; jj < 2; ++jj) st[nt].o[jj] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int w2 = 0; w2 < 4; ++w2) {
            // a wavefront that saw no tile of a row left m = -inf and sums of zero for it
            const float a = ml[w2].x == -INFINITY ? 0.0f : __builtin_amdgcn_exp2f(ml[w2].x - mx);
            st[nt].l += a * ml[w2].y;
#pragma unroll
            for (int jj = 0; jj < 2; ++jj) st[nt].o[jj] += a * o[w2][jj];
        }
    }
    if constexpr (SPLIT)
        if (!fold_slices<NT, 2, 8>(plan.split, slice, n_kv, kvh, wave, 1, lane, st, j0)) return;
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) write(std::integral_constant<int, 2>{}, j0, nt);
}

// (Two wavefronts per SIMD: declared for one, the compiler keeps accumulators in the other register file and copies them per tile.)
// Where the tables are: on the device, or the kernel's first argument, packed or not.
enum FewFrom { kFewDevice, kFewArguments, kFewPacked };
template <int NT, bool F8, bool SPLIT, int FROM>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2))) void attention_bf16_few(
    PlanWords<FROM != kFewDevice>, const char* __restrict__ pool, const uint16_t* __restrict__ q, PlanDev plan, int n_cand, int n_q, int n_kv,
    int group, float scale_log2e, PartialBuf part, const uint16_t* __restrict__ cand_k, const uint16_t* __restrict__ cand_v,
    const uint8_t* __restrict__ cand_mask, uint16_t* __restrict__ out) {
    __shared__ __attribute__((aligned(16))) char lds[FewLds<NT>::kBytes];
    const Slice slice = unit_of_block<SPLIT, FROM != kFewDevice>(plan, 0, n_kv);
    tables_unwritten(plan);
    attend_few<NT, F8, SPLIT, FROM == kFewPacked>(lds, slice, pool, q, plan, n_cand, n_q, n_kv, group, scale_log2e, part, cand_k, cand_v, cand_mask, out);
}

}  // namespace

// Lays the tables of inline_words out packed, in the order descriptors, blocks, tiles, threads; false if they do not fit.
static bool pack_tables(PlanDev& plan, PlanWords<true>& to) {
    const char* from = (const char*)plan.inline_words;
    const size_t bytes = (size_t)plan.n_inline_words * 4, tiles_at = (size_t)plan.tiles, threads_at = (size_t)plan.dfs_threads;
    size_t n_blocks = 0;
    for (int k = 0; k < 3; ++k) n_blocks += (size_t)plan.split.n_blocks_class[k];
    if (threads_at > bytes || tiles_at > threads_at) return false;
    const size_t n_wg = (size_t)plan.n_wg, n_tiles = (threads_at - tiles_at) / sizeof(TileRef), n_threads = (bytes - threads_at) / 4;
    if (few_packed_words(n_wg, n_blocks, n_tiles, n_threads) > (size_t)kPlanInlineWords) return false;
    uint32_t* at = (uint32_t*)to.words;
    const WgDesc* wgs = (const WgDesc*)(from + (size_t)plan.wgs);
    plan.wgs = nullptr;  // (offsets from here on)
    for (size_t g = 0; g < n_wg; ++g)
        for (int k = 0; k < 4; ++k, at += kFewWaveWords) {
            uint32_t w[kFewWaveWords];
            pack_few_wave(wgs[g].w[k], wgs[g].n_full[k], w);
            memcpy(at, w, sizeof w);
        }
    const char* blocks = from + (size_t)plan.split.blocks;
    plan.split.blocks = (const SplitBlock*)((char*)at - (char*)to.words);
    memcpy(at, blocks, n_blocks * sizeof(SplitBlock));
    at += n_blocks * sizeof(SplitBlock) / 4;
    const TileRef* tiles = (const TileRef*)(from + tiles_at);
    plan.tiles = (const TileRef*)((char*)at - (char*)to.words);
    for (size_t i = 0; i < n_tiles; ++i) *at++ = pack_few_tile(tiles[i]);
    plan.dfs_threads = (const int32_t*)((char*)at - (char*)to.words);
    memcpy(at, from + threads_at, n_threads * 4);
    return true;
}

hipError_t launch_attention_few_bf16(const Shape& s, const void* pool, const void* q, const PlanDev& staged, int n_cand, PartialBuf part,
                                     const void* cand_k, const void* cand_v, const uint8_t* mask, void* out, hipStream_t st) {
    PlanDev plan = staged;
    if (plan.few != 2 && plan.n_inline_words > kPlanInlineWords) return hipErrorInvalidValue;
    const bool split = plan.split.blocks != nullptr || plan.inline_words;
    const int32_t* n_class = split ? plan.split.n_blocks_class : plan.n_wg_class;
    const int64_t n_wg = ((int64_t)n_class[1] + n_class[2]) * s.n_kv;
    if (n_class[0] > 0 || n_wg > 0x7fffffff) return hipErrorInvalidValue;
    if (n_wg == 0) return hipSuccess;
#define APAR_LAUNCH(KERNEL, WORDS)                                                                           \
    hipLaunchKernelGGL(KERNEL, dim3((unsigned)n_wg), dim3(256), 0, st, WORDS, (const char*)pool,             \
                       (const uint16_t*)q, plan, n_cand, s.n_q, s.n_kv, s.group, s.scale_log2e, part,        \
                       (const uint16_t*)cand_k, (const uint16_t*)cand_v, mask, (uint16_t*)out)
#define APAR_LAUNCH_NT(F8V, SPLITV, FROMV, WORDS)                                                         \
    do {                                                                                                     \
        if (n_class[1] > 0) APAR_LAUNCH((attention_bf16_few<2, F8V, SPLITV, FROMV>), WORDS);               \
        else APAR_LAUNCH((attention_bf16_few<1, F8V, SPLITV, FROMV>), WORDS);                              \
    } while (0)
#define APAR_LAUNCH_F8(SPLITV, FROMV, WORDS)                                                               \
    do {                                                                                                     \
        if (s.fp8_sealed) APAR_LAUNCH_NT(true, SPLITV, FROMV, WORDS);                                      \
        else APAR_LAUNCH_NT(false, SPLITV, FROMV, WORDS);                                                  \
    } while (0)
    if (plan.inline_words) {
        PlanWords<true> words;
        if (plan.few == 2) {
            if (!pack_tables(plan, words)) return hipErrorInvalidValue;
            APAR_LAUNCH_F8(true, kFewPacked, words);
        } else {
            memcpy(words.words, plan.inline_words, (size_t)plan.n_inline_words * sizeof(int32_t));
            APAR_LAUNCH_F8(true, kFewArguments, words);
        }
    } else if (split) {
        APAR_LAUNCH_F8(true, kFewDevice, PlanWords<false>{});
    } else {
        APAR_LAUNCH_F8(false, kFewDevice, PlanWords<false>{});
    }
#undef APAR_LAUNCH_F8
#undef APAR_LAUNCH_NT
#undef APAR_LAUNCH
    return hipGetLastError();
}

}  // namespace apar
