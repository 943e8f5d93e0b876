// Decode attention over fp32 KV tiles (row-major, 16 token slots of D floats, K then V) on the gfx950 matrix
// cores: v_mfma_f32_16x16x4_f32, whose products and sums are IEEE fp32 throughout.
//
// The same plan and the same mapping as the bf16 kernel: query rows on the N side of 16x16 tiles, the token
// slots of a block on the M side,
//
//   S^T[token][row] = K[token][:] . Q[row][:]            D / 4 products of 4 dims
//   O^T[dim][row]  += V^T[dim][token] . P^T[token][row]   4 x D / 16 products of 4 tokens
//
// with both contractions taken in an order in which a lane's operands are runs of a row as it lies in memory.
// With lane = 16 g + c (J = D / 16):
//   K, Q: lane holds dims 16 j + 4 g .. + 3 of token / row c, j < J; product (j, i) contracts dims 16 j + 4 g + i
//   V:    lane holds dims J c .. J c + J - 1 of tokens 4 g .. 4 g + 3; product (jj, i) contracts tokens 4 g + i into
//         dims J m + jj
//   S:    lane holds the logits of tokens 4 g + i of row c, which is the operand layout of P (no lane exchange)
//   O:    lane holds dims J (4 g + i) + jj of row c: 4 J consecutive ones
// so every load is 16 bytes per lane, no value moves between lanes and nothing is staged: a tile goes from
// memory to operand registers, K refilled after the K.Q^T products, V after the V^T.P^T products, for the tiles
// of the shared list as for a wavefront's own (the four wavefronts of a workgroup meet in the caches).
// What bounds it: the fp32 matrix rate (a tile of D = 128 is 64 products of 32 cycles for 16 KiB) where rows
// share blocks, else memory; with few threads the chain of tiles of the longest unit.
// Measured against one wavefront per query row in plain vector arithmetic, every row reading its blocks for
// itself: twelve depth-2 trees (32 / 8 heads, d = 128, 0.28 GB read) 704 -> 355 us; one request of three
// threads (2 heads, d = 64) 56 -> 16 us for the call; error against 64 bits 5.2e-7 -> 4.5e-7 and 2.2e-7 -> 1.9e-7.
// With its heaviest units cut into slices (attn_split.hpp) the first of these took 137 us, in one launch 94, and in units of 16
// rows without shared lists, as the plans of such calls have them now (PlanParams::few_units), 77; one request of five threads,
// 8 kv heads 26.3 -> 12.5, of 14 k tokens and 30 threads of four candidates 91 -> 54, three of five candidates 117 -> 28.
//
// A row that does not see a block meets it with probability 0, and 0 times an infinity or a NaN is a NaN.  Blocks of
// other threads must not do that to a row: a wavefront takes those of its rows that did not come out finite again, one
// by one, over the blocks each of them sees.
#include <hip/hip_runtime.h>

#include <cstring>

#include "apar_internal.hpp"
#include "attn_split.hpp"

namespace apar {

namespace {

typedef __attribute__((__vector_size__(4 * sizeof(float)))) float f32x4;

constexpr float kSlack = 8.0f;  // a probability may exceed 1 by at most 2^kSlack before the reference moves

__device__ __forceinline__ float wave_sum(float x) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) x += __shfl_xor(x, o, 64);
    return x;
}

template <int D>
struct Row {  // the 16 rows of one tile: query operands and running softmax state
    f32x4 q[D / 16];
    f32x4 o[D / 16];
    float m, l;
};

template <int D>
__device__ __forceinline__ f32x4 products(const f32x4 (&k)[D / 16], const Row<D>& st) {
    // four chains: a quarter of the latency, and sums of a quarter of the length (twelve trees, two chains / four: error against
    // 64 bits 3.4e-7 / 2.9e-7, three threads 2.1e-7 / 1.6e-7; the eight additions more are 2 to 3 % of a call that is bound by products at
    // d = 64 and 1 % at d = 128, prefill of segments for example)
    f32x4 a[4];
#pragma unroll
    for (int h = 0; h < 4; ++h) a[h] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int j = 0; j < D / 16; j += 4)
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int h = 0; h < 4; ++h) a[h] = __builtin_amdgcn_mfma_f32_16x16x4f32(k[j + h][i], st.q[j + h][i], a[h], 0, 0, 0);
    return (a[0] + a[1]) + (a[2] + a[3]);
}

// tok_mask: the token slots this lane's row sees (none: not its block).
__device__ __forceinline__ f32x4 masked(const f32x4& s, uint32_t tok_mask, int g4) {
    const uint32_t mine = tok_mask >> (4 * g4);
    f32x4 x;
#pragma unroll
    for (int i = 0; i < 4; ++i) x[i] = ((mine >> i) & 1u) ? s[i] : -INFINITY;
    return x;
}

// One tile's logits, -inf where this lane's row does not see the token, into one row tile's state.
template <int D>
__device__ __forceinline__ void accumulate(const f32x4 (&v)[4][D / 64], Row<D>& st, const f32x4& x, float scale_log2e) {
    constexpr int J = D / 16;
    const float top = fmaxf(fmaxf(x[0], x[1]), fmaxf(x[2], x[3])) * scale_log2e;
    if (__builtin_amdgcn_ballot_w64(top > st.m + kSlack) != 0) {
        // some row ran away from its reference: every row's moves to its running maximum (its four lanes agree on it)
        float mx = fmaxf(top, __shfl_xor(top, 16, 64));
        mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
        const float m_new = fmaxf(st.m, mx);
        const float alpha = (m_new == -INFINITY) ? 1.0f : __builtin_amdgcn_exp2f(st.m - m_new);
        st.l *= alpha;
#pragma unroll
        for (int jj = 0; jj < J; ++jj) st.o[jj] *= alpha;
        st.m = m_new;
    }
    const float bias = st.m != -INFINITY ? -st.m : -INFINITY;  // (a row that has seen nothing yet)
    float p[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) p[i] = __builtin_amdgcn_exp2f(__builtin_fmaf(x[i], scale_log2e, bias));
    st.l += (p[0] + p[1]) + (p[2] + p[3]);
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int jj = 0; jj < J; ++jj)
            st.o[jj] = __builtin_amdgcn_mfma_f32_16x16x4f32(v[i][jj / 4][jj % 4], p[i], st.o[jj], 0, 0, 0);
}

// NT = 16-row tiles per wavefront; SPLIT: several workgroups per unit, each with a slice of its lists (attn_split.hpp).
// lds: three wavefronts' row states when a unit is split; one wavefront's rows each when rows are taken again one by one
template <int D, int NT, bool SPLIT>
__device__ __forceinline__ void attend_unit(float (&lds)[4][16 * D + 32], const Slice& slice, const char* __restrict__ pool,
                                            const float* __restrict__ q, const PlanDev& plan, int n_cand, int n_q, int n_kv, int group,
                                            float scale_log2e, const PartialBuf& part, const float* __restrict__ cand_k,
                                            const float* __restrict__ cand_v, const uint8_t* __restrict__ cand_mask, float* __restrict__ out) {
    constexpr int J = D / 16;
    constexpr int kTile = 2 * 16 * D * 4;  // bytes of one (block, kv head)
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int g4 = lane >> 4, c = lane & 15;
    const int kvh = blockIdx.x % n_kv;
    const WgDesc* wg = plan.wgs + slice.wg;
    WaveItem wi = wg->w[wave];
    if (wi.n_grp == 0) return;  // (a wave-split unit's wavefronts all have rows; nobody waits for this one)
    int coop_ofs = wg->coop_ofs, n_coop = wg->n_coop, n_full = 0;
    if constexpr (SPLIT) {
        cut_list(slice, coop_ofs, n_coop, n_full);
        cut_list(slice, wi.tile_ofs, wi.n_tiles, n_full);
    }
    const char* head_base = pool + (int64_t)kvh * kTile;
    const int64_t block_stride = (int64_t)n_kv * kTile;

    // Row geometry: column c of row tile nt is row `within` of the wavefront's row group nt * cap + c / rps.
    const int rps = plan.rows_per_slice, n_sl = plan.n_slices, rpt = plan.rows_per_thread;
    const int cap = 16 / rps;
    auto row_of = [&](int nt, int col, int& j, int& listed, int& cc, int64_t& qrow, int64_t& slot) -> bool {
        const int jc = col / rps, within = col - jc * rps;
        j = nt * cap + jc;
        const int grp = wi.grp_lo + j;
        const int rank = grp / n_sl, rr = (grp - rank * n_sl) * rps + within;
        if (jc >= cap || j >= wi.n_grp || rr >= rpt) return false;
        listed = plan.dfs_threads ? plan.dfs_threads[rank] : rank;
        cc = rr / group;
        const int hq = kvh * group + (rr - cc * group);
        qrow = ((int64_t)listed * n_cand + cc) * n_q + hq;
        slot = ((int64_t)(wi.part_base + rank - wi.grp_lo / n_sl) * n_cand + cc) * n_q + hq;
        return true;
    };
    Row<D> st[NT];
    int my_j[NT];  // row group of this lane's row, relative to the wavefront's first; -1: no row
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
        int j, listed, cc;
        int64_t qrow, slot;
        const bool ok = row_of(nt, c, j, listed, cc, qrow, slot);
        my_j[nt] = ok ? j : -1;
        st[nt].m = -INFINITY;
        st[nt].l = 0.0f;
#pragma unroll
        for (int jj = 0; jj < J; ++jj) {
            st[nt].o[jj] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
            st[nt].q[jj] = ok ? *reinterpret_cast<const f32x4*>(q + qrow * D + 16 * jj + 4 * g4) : f32x4{0.0f, 0.0f, 0.0f, 0.0f};
        }
    }
    // how many of a tile's tokens the row `ahead` row groups past its first one sees (causal tiles: one more per group)
    auto seen = [](int meta, int ahead) -> int {
        const int fill = (meta >> 20) & 31;
        return (meta >> 30) ? min(fill, max(0, ((meta >> 25) & 31) + ahead)) : fill;
    };

    f32x4 k[J], v[4][D / 64];
    // rows past the fill count hold anything: their lanes read row 0 again, under a probability of 0
    auto issue_k = [&](const TileRef& t) {
        const int fill = (t.meta >> 20) & 31;
        const float* p = reinterpret_cast<const float*>(head_base + t.blk * block_stride) + (c < fill ? c : 0) * D + 4 * g4;
#pragma unroll
        for (int j = 0; j < J; ++j) k[j] = *reinterpret_cast<const f32x4*>(p + 16 * j);
    };
    auto issue_v = [&](const TileRef& t) {
        const int fill = (t.meta >> 20) & 31;
        const float* p = reinterpret_cast<const float*>(head_base + t.blk * block_stride) + 16 * D + J * c;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int row = 4 * g4 + i < fill ? 4 * g4 + i : 0;
#pragma unroll
            for (int h = 0; h < D / 64; ++h) v[i][h] = *reinterpret_cast<const f32x4*>(p + row * D + 4 * h);
        }
    };
    // both lists, one after the other; `shift`: the shared list's ranges count row groups from the workgroup's first
    for (int list = 0; list < 2; ++list) {
        const TileRef* tiles = plan.tiles + (list == 0 ? coop_ofs : wi.tile_ofs);
        const int n = list == 0 ? n_coop : wi.n_tiles;
        const int shift = list == 0 ? wi.grp_lo - wg->grp_base : 0;
        // (tiles of the shared list that no row of this wavefront sees are passed over)
        auto next = [&](int t) {
            for (; t < n; ++t) {
                const int meta = tiles[t].meta;
                if ((meta & 1023) - shift < wi.n_grp && ((meta >> 10) & 1023) - shift > 0) break;
            }
            return t;
        };
        int t = next(0);
        if (t >= n) continue;
        TileRef cur = tiles[t];
        issue_k(cur);
        issue_v(cur);
        while (t < n) {
            t = next(t + 1);
            const TileRef nx = tiles[min(t, n - 1)];  // (past the end: the last tile once more, not used)
            const int lo = (cur.meta & 1023) - shift, hi = ((cur.meta >> 10) & 1023) - shift;
            f32x4 s[NT];
#pragma unroll
            for (int nt = 0; nt < NT; ++nt)
                if (NT == 1 || (lo < (nt + 1) * cap && hi > nt * cap)) s[nt] = products<D>(k, st[nt]);
            issue_k(nx);
#pragma unroll
            for (int nt = 0; nt < NT; ++nt)
                if (NT == 1 || (lo < (nt + 1) * cap && hi > nt * cap)) {
                    // (a count of tokens, not a mask: seven instructions less per row tile, prefill at d = 64 1 % faster)
                    const int mine = (my_j[nt] >= max(lo, 0) && my_j[nt] < hi ? seen(cur.meta, my_j[nt] - lo) : 0) - 4 * g4;
#pragma unroll
                    for (int i = 0; i < 4; ++i) s[nt][i] = i < mine ? s[nt][i] : -INFINITY;
                    accumulate<D>(v, st[nt], s[nt], scale_log2e);
                }
            issue_v(nx);
            cur = nx;
        }
    }
    // a multi-candidate call's candidates: one more tile of at most 8 token rows per thread, each visible to the rows
    // whose mask names it (the unit that writes the rows directly adds them)
    const bool with_cands = (wi.flags & kWaveDirect) && cand_mask != nullptr && (wave == 0 || !(wi.flags & kWaveSplit)) && slice.s == 0;
    if (with_cands) {
        const int64_t tok_stride = (int64_t)n_kv * D;
        for (int ru = wi.grp_lo / n_sl; ru <= (wi.grp_lo + wi.n_grp - 1) / n_sl; ++ru) {
            const int listed_u = plan.dfs_threads ? plan.dfs_threads[ru] : ru;
            const int64_t base = ((int64_t)listed_u * n_cand * n_kv + kvh) * D;
#pragma unroll
            for (int j = 0; j < J; ++j)
                k[j] = *reinterpret_cast<const f32x4*>(cand_k + base + (c < n_cand ? c : 0) * tok_stride + 16 * j + 4 * g4);
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int h = 0; h < D / 64; ++h)
                    v[i][h] = *reinterpret_cast<const f32x4*>(cand_v + base + (4 * g4 + i < n_cand ? 4 * g4 + i : 0) * tok_stride + J * c + 4 * h);
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) {
                uint32_t tm = 0;
                int j, listed, cc;
                int64_t qrow, slot;
                if (row_of(nt, c, j, listed, cc, qrow, slot) && (wi.grp_lo + j) / n_sl == ru)
                    tm = cand_mask[(int64_t)listed_u * n_cand + cc] & ((1u << n_cand) - 1u);
                if (__builtin_amdgcn_ballot_w64(tm != 0) == 0) continue;
                accumulate<D>(v, st[nt], masked(products<D>(k, st[nt]), tm, g4), scale_log2e);
            }
        }
    }

    // ---- rows that did not come out finite, one by one ------------------------------------------
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
        bool fine = fabsf(st[nt].l) < INFINITY;
#pragma unroll
        for (int jj = 0; jj < J; ++jj)
#pragma unroll
            for (int i = 0; i < 4; ++i) fine = fine && fabsf(st[nt].o[jj][i]) < INFINITY;
        const uint64_t off = __builtin_amdgcn_ballot_w64(my_j[nt] >= 0 && !fine);
        if (off == 0) continue;
        const uint32_t bad = (uint32_t)(off | off >> 16 | off >> 32 | off >> 48) & 0xffffu;  // by column: any of a row's four lanes
        float* rows = lds[wave];
        for (int col = 0; col < 16; ++col) {
            int j, listed, cc;
            int64_t qrow, slot;
            if (!((bad >> col) & 1u) || !row_of(nt, col, j, listed, cc, qrow, slot)) continue;
            constexpr int E = D / 64;
            float qv[E], acc[E], m = -INFINITY, l = 0.0f;
#pragma unroll
            for (int e = 0; e < E; ++e) qv[e] = q[qrow * D + lane + 64 * e], acc[e] = 0.0f;
            auto take = [&](const float* krow, const float* vrow) {
                float dot = 0.0f;
#pragma unroll
                for (int e = 0; e < E; ++e) dot += qv[e] * krow[lane + 64 * e];
                const float sc = wave_sum(dot) * scale_log2e;
                const float m_new = fmaxf(m, sc);
                // a logit of -inf weighs nothing, also before any other (a NaN stays one, through pr)
                const float alpha = m_new == -INFINITY ? 1.0f : exp2f(m - m_new), pr = sc == -INFINITY ? 0.0f : exp2f(sc - m_new);
                l = l * alpha + pr;
#pragma unroll
                for (int e = 0; e < E; ++e) acc[e] = acc[e] * alpha + pr * vrow[lane + 64 * e];
                m = m_new;
            };
            for (int list = 0; list < 2; ++list) {
                const TileRef* tiles = plan.tiles + (list == 0 ? coop_ofs : wi.tile_ofs);
                const int n = list == 0 ? n_coop : wi.n_tiles;
                const int jl = list == 0 ? j + (wi.grp_lo - wg->grp_base) : j;
                for (int t = 0; t < n; ++t) {
                    const int meta = tiles[t].meta, lo = meta & 1023, hi = (meta >> 10) & 1023;
                    if (jl < lo || jl >= hi) continue;
                    const float* tile = reinterpret_cast<const float*>(head_base + tiles[t].blk * block_stride);
                    const int n_seen = seen(meta, jl - lo);
                    for (int tok = 0; tok < n_seen; ++tok) take(tile + tok * D, tile + (16 + tok) * D);
                }
            }
            if (with_cands) {
                const uint32_t bits = cand_mask[(int64_t)listed * n_cand + cc];
                for (int cp = 0; cp < n_cand; ++cp)
                    if ((bits >> cp) & 1u) {
                        const int64_t base = (((int64_t)listed * n_cand + cp) * n_kv + kvh) * D;
                        take(cand_k + base, cand_v + base);
                    }
            }
#pragma unroll
            for (int e = 0; e < E; ++e) rows[col * D + lane + 64 * e] = acc[e];
            if (lane == 0) rows[16 * D + 2 * col] = m, rows[16 * D + 2 * col + 1] = l;
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        if ((bad >> c) & 1u) {
#pragma unroll
            for (int jj = 0; jj < J; ++jj)
#pragma unroll
                for (int i = 0; i < 4; ++i) st[nt].o[jj][i] = rows[c * D + (4 * g4 + i) * J + jj];
            st[nt].m = rows[16 * D + 2 * c];
            st[nt].l = g4 == 0 ? rows[16 * D + 2 * c + 1] : 0.0f;  // the four lanes of a row add up to its sum
        }
        __builtin_amdgcn_wave_barrier();
    }

    // ---- results --------------------------------------------------------------------------------
    if (NT == 1 && (wi.flags & kWaveSplit)) {
        // the four wavefronts hold the same rows over different tiles: fold 1..3 into 0 through LDS
        Row<D>& s0 = st[0];
        float lt = s0.l;
        lt += __shfl_xor(lt, 16, 64);
        lt += __shfl_xor(lt, 32, 64);
        if (wave > 0) {
#pragma unroll
            for (int jj = 0; jj < J; ++jj) *reinterpret_cast<f32x4*>(&lds[wave][(jj * 64 + lane) * 4]) = s0.o[jj];
            if (g4 == 0) lds[wave][16 * D + 2 * c] = s0.m, lds[wave][16 * D + 2 * c + 1] = lt;
        }
        __syncthreads();
        if (wave > 0) return;
        float mx = s0.m;
        for (int w2 = 1; w2 < 4; ++w2) mx = fmaxf(mx, lds[w2][16 * D + 2 * c]);
        // a wavefront that saw no tile of a row left m = -inf and sums of zero for it
        const float a0 = (s0.m == -INFINITY) ? 0.0f : __builtin_amdgcn_exp2f(s0.m - mx);
        if (s0.m != -INFINITY) {
            lt *= a0;
#pragma unroll
            for (int jj = 0; jj < J; ++jj) s0.o[jj] *= a0;
        }
        for (int w2 = 1; w2 < 4; ++w2) {
            const float mw = lds[w2][16 * D + 2 * c];
            if (mw == -INFINITY && lds[w2][16 * D + 2 * c + 1] == 0.0f) continue;
            const float aw = __builtin_amdgcn_exp2f(mw - mx);
            lt += aw * lds[w2][16 * D + 2 * c + 1];
#pragma unroll
            for (int jj = 0; jj < J; ++jj) s0.o[jj] += aw * *reinterpret_cast<const f32x4*>(&lds[w2][(jj * 64 + lane) * 4]);
        }
        s0.m = mx;
        s0.l = g4 == 0 ? lt : 0.0f;
    }
    if constexpr (SPLIT)
        if (!fold_slices<NT, J>(plan.split, slice, n_kv, kvh, wave, (wi.flags & kWaveSplit) ? 1 : 4, lane, st)) return;
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
        float lt = st[nt].l;
        lt += __shfl_xor(lt, 16, 64);
        lt += __shfl_xor(lt, 32, 64);
        int j, listed, cc;
        int64_t qrow, slot;
        if (!row_of(nt, c, j, listed, cc, qrow, slot)) continue;
        const bool direct = (wi.flags & kWaveDirect) != 0;
        const float inv = direct ? 1.0f / lt : 1.0f;
        float* dst = direct ? out + qrow * D : part.o + slot * D;
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int h = 0; h < J / 4; ++h) {
                const f32x4 x = {st[nt].o[4 * h][i] * inv, st[nt].o[4 * h + 1][i] * inv, st[nt].o[4 * h + 2][i] * inv, st[nt].o[4 * h + 3][i] * inv};
                *reinterpret_cast<f32x4*>(dst + (4 * g4 + i) * J + 4 * h) = x;
            }
        if (!direct && g4 == 0) {
            part.ml[slot * 2] = st[nt].m;
            part.ml[slot * 2 + 1] = lt;
        }
    }
}

// Units of either row-tile class, in one launch (one launch after the other: twelve trees, 8 kv heads 118 -> 94 us, eight of 300
// rows, group 8, 111 -> 79, four candidates 96 -> 63).  It holds as many wavefronts as the two-tile class needs registers for: two per
// SIMD (d = 128) or three (d = 64), where the one-tile class alone would have three at most and four.  Calls of that class do not
// gain by a kernel of their own (us, by it / by this one; workgroups): d = 64 (3008) 131 / 130, (1576) 102 / 103, (1200) 24.3 / 25.0,
// (768) 63.5 / 63.5, 100 requests of two fork levels 79 / 71; d = 128 (3008) 254 / 253, (1576) 195 / 195, (480) 56 / 56, (192) 47 / 47: their
// wavefronts are busy with products.  INLINE (with SPLIT): the plan's tables come with the kernel's arguments.
template <int D, bool SPLIT, bool INLINE>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2))) void attention_f32(
    PlanWords<INLINE>, const char* __restrict__ pool, const float* __restrict__ q, PlanDev plan, int n_cand, int n_q, int n_kv,
    int group, float scale_log2e, PartialBuf part, const float* __restrict__ cand_k, const float* __restrict__ cand_v,
    const uint8_t* __restrict__ cand_mask, float* __restrict__ out) {
    __shared__ __attribute__((aligned(16))) float lds[4][16 * D + 32];
    if constexpr (INLINE) plan_from_arguments(plan);
    Slice slice;
    if constexpr (SPLIT) {
        slice = slice_of_block(plan.split, 0, n_kv);
    } else {
        slice.wg = blockIdx.x / n_kv;
    }
    tables_unwritten(plan);
    if ((plan.wgs[slice.wg].row_tiles & 255) == 2)
        attend_unit<D, 2, SPLIT>(lds, slice, pool, q, plan, n_cand, n_q, n_kv, group, scale_log2e, part, cand_k, cand_v, cand_mask, out);
    else
        attend_unit<D, 1, SPLIT>(lds, slice, pool, q, plan, n_cand, n_q, n_kv, group, scale_log2e, part, cand_k, cand_v, cand_mask, out);
}

}  // namespace

hipError_t launch_attention_f32(const Shape& s, const void* pool, const void* q, const PlanDev& plan, int n_cand, PartialBuf part,
                                const void* cand_k, const void* cand_v, const uint8_t* mask, void* out, hipStream_t st) {
    if (plan.n_inline_words > kPlanInlineWords) return hipErrorInvalidValue;
    const bool split = plan.split.blocks != nullptr || plan.inline_words;
    const int32_t* n_class = split ? plan.split.n_blocks_class : plan.n_wg_class;
    const int64_t n = ((int64_t)n_class[1] + n_class[2]) * s.n_kv;
    if (n > 0x7fffffff || n_class[0] > 0) return hipErrorInvalidValue;  // (fp32 pools have no matrix units)
    if (n == 0) return hipSuccess;
#define APAR_LAUNCH(DV, SPLITV, INLINEV, WORDS)                                                                           \
    hipLaunchKernelGGL((attention_f32<DV, SPLITV, INLINEV>), dim3((unsigned)n), dim3(256), 0, st, WORDS,                  \
                       (const char*)pool, (const float*)q, plan, n_cand, s.n_q, s.n_kv, s.group, s.scale_log2e,           \
                       part, (const float*)cand_k, (const float*)cand_v, mask, (float*)out)
#define APAR_LAUNCH_D(SPLITV, INLINEV, WORDS)                \
    do {                                                     \
        if (s.d == 64) APAR_LAUNCH(64, SPLITV, INLINEV, WORDS); \
        else APAR_LAUNCH(128, SPLITV, INLINEV, WORDS);       \
    } while (0)
    if (plan.inline_words) {
        PlanWords<true> words;
        memcpy(words.words, plan.inline_words, (size_t)plan.n_inline_words * sizeof(int32_t));
        APAR_LAUNCH_D(true, true, words);
    } else if (split) {
        APAR_LAUNCH_D(true, false, PlanWords<false>{});
    } else {
        APAR_LAUNCH_D(false, false, PlanWords<false>{});
    }
#undef APAR_LAUNCH_D
#undef APAR_LAUNCH
    return hipGetLastError();
}

}  // namespace apar
