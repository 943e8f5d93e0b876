// Decode attention over bf16 KV tiles on the gfx950 matrix cores.
//
// Query rows - (thread, candidate, q head of one kv group) - sit on the N side
// of 16x16 matrix-core tiles, the 16 token slots of a block on the M side:
//
//   S^T[token][row] = K[token][:] . Q[row][:]          4 x mfma_f32_16x16x32_bf16
//   O^T[dim][row]  += V^T[dim][token] . P^T[token][row] 8 x mfma_f32_16x16x16_bf16
//
// K and V^T are the A operands and are stored in HBM in operand order (see the
// layout note in apar_internal.hpp): a wavefront fetches a tile half with four
// 16-byte loads per lane, each a contiguous 1 KiB.  The accumulator layout of
// S^T (lane = 16*g + c holds tokens 4g..4g+3 of row c) is already the
// B-operand layout of P^T, so probabilities never move between lanes.
//
// A workgroup (4 wavefronts, 16 or 32 rows each) is given by the host plan
//   * a shared tile list: blocks whose holders sit in more than one wavefront
//     (prefixes shared by many sibling threads).  They go through LDS in groups
//     of four, one whole tile per wavefront, the next group in flight to
//     registers while the current one is consumed (two barriers per group), and
//     every wavefront applies each tile to those of its rows that hold the block;
//   * one private tile list per wavefront: blocks held only by rows of that
//     wavefront (private tails, small sibling groups), loaded straight from HBM
//     into operand registers with no barrier.  K registers are refilled right
//     after the K.Q^T products and V registers after the V^T.P^T products, so
//     the next tile is in flight while the current one is consumed.
// Every list holds its full tiles first: they run through loops with nothing
// but unconditional loads; the open tiles after them through general loops.
// Every tile names the range of row groups it applies to; other rows see -inf
// logits.  A causal tile (prefill: the query tokens are the row groups) shows
// each further row group one more of its token slots.  A row's softmax state stays in registers across all the blocks of
// its root path that the unit covers; attention is a set operation, so the
// order in which a unit visits them does not matter.  Rows whose whole path
// lies in the unit are normalised and written out here; the others leave a
// partial result (reference, sum, unnormalised output) for the merge kernel.
//
// A block that is still filling (fewer than 16 slots) is stored row-major, not in
// operand order; such tiles - at most one per segment - take a slower path: K
// pieces are gathered row by row and V goes through a padded LDS transpose.
//
// fp8 pools (template parameter F8): a full block holds fp8 codes in the same element order, half the
// bytes, and one power-of-two scale per half.  Its tiles are fetched with two 16-byte loads per lane and
// half and turned into the bf16 operands by the hardware conversion that multiplies by the scale (exact: a
// code times a power of two is a bf16 value) - private tiles on their way into the operand registers,
// shared tiles once, by the wavefront that stages them, so that LDS holds the bf16 tile.  Everything after
// that - products, softmax, accumulation - is the code of the bf16 pool.
// Blocks that are still filling are bf16 rows on either pool.
//
// Softmax runs in base 2 with a lazily updated reference: a row's reference
// logit m only moves when some logit exceeds it by more than kSlack, which
// keeps the cross-lane maximum and the rescale of the accumulators off the
// common path.
#include <hip/hip_runtime.h>

#include <cstring>
#include <type_traits>

#include "attn_bf16.hpp"

namespace apar {

namespace {

// NT = 16-row tiles per wavefront (1 or 2 are instantiated): a workgroup carries up to 64 * NT query rows.
// F8: full blocks hold fp8 codes and two scales (APAR_BF16_FP8KV pools).
// SPLIT: several workgroups per unit, each with a slice of its tile lists (attn_split.hpp).
// lds: four staged tiles during the shared phase; then one V-transpose scratch per wavefront; last, three wavefronts' row
// states when a unit is split
constexpr int kAttnLds = 4 * kTileBytes;
static_assert(kAttnLds >= 3 * kSplitState && kAttnLds >= 4 * kOpenScratch && kOpenRowStride >= 256, "LDS areas overlap in time");
template <int NT, bool F8, bool SPLIT>
__device__ __forceinline__ void attend_unit(char* lds, const Slice& slice, const char* __restrict__ pool, const uint16_t* __restrict__ q,
                                            const PlanDev& plan, int n_cand, int n_q, int n_kv, int group, float scale_log2e,
                                            const PartialBuf& part, const uint16_t* __restrict__ cand_k,
                                            const uint16_t* __restrict__ cand_v, const uint8_t* __restrict__ cand_mask,
                                            uint16_t* __restrict__ out) {
    char(*stage)[kTileBytes] = reinterpret_cast<char(*)[kTileBytes]>(lds);
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int g4 = lane >> 4, c = lane & 15;
    const int kvh = blockIdx.x % n_kv;
    const WgDesc* wg = plan.wgs + slice.wg;
    WaveItem wi = wg->w[wave];
    int n_coop = wg->n_coop, coop_ofs = wg->coop_ofs, coop_full = wg->row_tiles >> 8;
    int own_full = min(wg->n_full[wave], wi.n_tiles);
    if constexpr (SPLIT) {
        cut_list(slice, coop_ofs, n_coop, coop_full);
        cut_list(slice, wi.tile_ofs, wi.n_tiles, own_full);
    }
    const TileRef* coop = plan.tiles + coop_ofs;
    const TileRef* mine = plan.tiles + wi.tile_ofs;
    const char* head_base = pool + (int64_t)kvh * kTileBytes;
    const int64_t block_stride = (int64_t)n_kv * kTileBytes;

    // Row geometry: column c of row tile nt is row `within` of the wavefront's row group nt * cap + c / rps.
    const int rps = plan.rows_per_slice, n_sl = plan.n_slices, rpt = plan.rows_per_thread;
    const int cap = 16 / rps;
    const int jc = c / rps, within = c - jc * rps;
    RowState st[NT];
    int my_j[NT];       // row group of this lane's row, relative to the wavefront's first; 0x7fff: no row
    // where the row of tile nt lives: depth-first rank of its thread, row within the thread's rows,
    // q/output row and partial-result slot (recomputed where needed rather than kept in registers)
    auto locate = [&](int nt, int& rank, int& rr, int64_t& qrow, int64_t& slot) {
        const int grp = wi.grp_lo + nt * cap + jc;
        rank = grp / n_sl;
        rr = (grp - rank * n_sl) * rps + within;
        const int listed = plan.dfs_threads ? plan.dfs_threads[rank] : rank;
        const int cc = rr / group, hq = kvh * group + (rr - cc * group);
        qrow = ((int64_t)listed * n_cand + cc) * n_q + hq;
        slot = ((int64_t)(wi.part_base + rank - wi.grp_lo / n_sl) * n_cand + cc) * n_q + hq;
    };
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
        const int j = nt * cap + jc;
        const int grp = wi.grp_lo + j;
        const int rank = grp / n_sl, rr = (grp - rank * n_sl) * rps + within;
        const bool ok = jc < cap && j < wi.n_grp && rr < rpt;
        my_j[nt] = ok ? j : 0x7fff;
        st[nt].m = -INFINITY;
        st[nt].l = 0.0f;
#pragma unroll
        for (int kk = 0; kk < 4; ++kk) st[nt].q[kk].u = u32x4{0u, 0u, 0u, 0u};
#pragma unroll
        for (int jj = 0; jj < 8; ++jj) st[nt].o[jj] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
        if (ok) {
            int rk, r2;
            int64_t qrow, slot;
            locate(nt, rk, r2, qrow, slot);
            const u32x4* qp = reinterpret_cast<const u32x4*>(q + qrow * 128 + g4 * 32);
#pragma unroll
            for (int kk = 0; kk < 4; ++kk) st[nt].q[kk].u = qp[kk];
        }
    }
    // token slots of a tile that the row `ahead` row groups past the tile's first one may see: the filled
    // ones; of a causal tile (bit 30) `first` slots (bits 25-29) for the first row group and one more for
    // every further one
    auto visible = [](int meta, int ahead) -> uint32_t {
        const int fill = (meta >> 20) & 31;
        const int limit = (meta >> 30) ? min(fill, max(0, ((meta >> 25) & 31) + ahead)) : fill;
        return (1u << limit) - 1u;
    };
    // does a tile touch row tile nt at all?  (wavefront-uniform)
    auto touches = [&](int nt, int lo, int hi) -> bool {
        return lo < min((nt + 1) * cap, wi.n_grp) && hi > nt * cap;
    };

    // Makes the query operands' loads known to have landed (an empty statement that names the registers:
    // the compiler must wait for them there).  Used once in front of the shared-tile loops.  Without it the
    // compiler's wait-count bookkeeping carries the query loads of the kernel's start into those loops as
    // if they were the youngest loads in flight, and every product waits for the tile prefetch issued just
    // before it, which defeats the prefetch.
    auto settle_queries = [&]() {
#pragma unroll
        for (int nt = 0; nt < NT; ++nt)
#pragma unroll
            for (int kk = 0; kk < 4; ++kk) asm("" : "+v"(st[nt].q[kk].u));
    };

    // ---- shared tiles: staged once in LDS for the whole workgroup ---------------------------
    // Tiles go through LDS in groups of four, one whole tile per wavefront: while a group is consumed
    // from LDS, each wavefront already has its tile of the next group in flight to its registers.
    // Full tiles (16 filled slots) come first in every list and go through a loop that contains no
    // lane-dependent branch around a load (which would make the compiler wait for each load where it is
    // issued); the open tiles after them go through a general loop.
    if (n_coop > 0) {
        const int shift = wi.grp_lo - wg->grp_base;  // shared ranges are relative to the group's base
        const int n_coop_full = coop_full;
        u32x4 rk[4], rv[4];
        // Shared tiles are fetched with plain loads, private ones (below) with non-temporal loads: a shared
        // tile may be read again by another workgroup (the units below an inlined segment all read it; so do
        // the stand-alone units of a segment with many rows) and is worth a place in L2, a private tile is
        // read exactly once.  Measured: plain loads here take 6-10 % off the HBM traffic of the speculative
        // loop and 2 % off the headline launch; plain loads for the private tiles cost 8 %.
        f32x2 rsc = {1.0f, 1.0f};  // fp8 pools: the scales of the tile in flight
        auto fetch_full = [&](int t) {
            const char* tile = head_base + coop[t].blk * block_stride + lane * 16;
            if constexpr (F8) {
#pragma unroll
                for (int rp = 0; rp < 2; ++rp) {
                    rk[rp] = *reinterpret_cast<const u32x4*>(tile + rp * 1024);
                    rv[rp] = *reinterpret_cast<const u32x4*>(tile + kFp8HalfBytes + rp * 1024);
                }
                rsc = *reinterpret_cast<const f32x2*>(tile - lane * 16 + kFp8ScaleOfs);
            } else {
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    rk[r] = *reinterpret_cast<const u32x4*>(tile + r * 1024);
                    rv[r] = *reinterpret_cast<const u32x4*>(tile + 4096 + r * 1024);
                }
            }
        };
        auto fetch_any = [&](int t) {
            if (t >= n_coop) return;
            const int fill = (coop[t].meta >> 20) & 31;
            if (!F8 && fill == 16) {  // (a list holds its full tiles first: none of them comes through here on an fp8 pool)
                fetch_full(t);
            } else {
                // an open block is row-major: piece r of this lane belongs to token row 4r + g4.  Rows past the
                // fill count are never read: their lanes re-read row 0 instead (same cache lines, no extra
                // traffic, no branch around a load); the masked logits give those slots probability 0.
                const char* tile = head_base + coop[t].blk * block_stride + c * 16;
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int row = 4 * r + g4 < fill ? 4 * r + g4 : 0;
                    rk[r] = *reinterpret_cast<const u32x4*>(tile + row * 256);
                    rv[r] = *reinterpret_cast<const u32x4*>(tile + 4096 + row * 256);
                }
            }
        };
        auto to_stage = [&](auto full_tile) {
            char* dst = stage[wave] + lane * 16;
            if constexpr (F8 && decltype(full_tile)::value) {
                // the codes are widened once, by the wavefront that fetched them: what is staged is the bf16 tile in
                // operand order, as on a bf16 pool, and the four consumers read it as such
                Frag ks[4], vs[4];
                const u32x4 kraw[2] = {rk[0], rk[1]}, vraw[2] = {rv[0], rv[1]};
                fp8_operands(kraw, rsc.x, ks);
                fp8_operands(vraw, rsc.y, vs);
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    *reinterpret_cast<u32x4*>(dst + r * 1024) = ks[r].u;
                    *reinterpret_cast<u32x4*>(dst + 4096 + r * 1024) = vs[r].u;
                }
            } else {
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    *reinterpret_cast<u32x4*>(dst + r * 1024) = rk[r];
                    *reinterpret_cast<u32x4*>(dst + 4096 + r * 1024) = rv[r];
                }
            }
        };
        // the operands of a staged full tile
        auto staged_operands = [&](const char* sb, Frag (&ks)[4], Frag (&vs)[4]) {
#pragma unroll
            for (int r = 0; r < 4; ++r) ks[r].u = *reinterpret_cast<const u32x4*>(sb + r * 1024 + lane * 16);
#pragma unroll
            for (int r = 0; r < 4; ++r) vs[r].u = *reinterpret_cast<const u32x4*>(sb + 4096 + r * 1024 + lane * 16);
        };
        auto consume = [&](int t, const char* sb, auto full_only) {
            constexpr bool kFull = decltype(full_only)::value;
            const int meta = coop[t].meta;
            const int lo = (meta & 1023) - shift, hi = ((meta >> 10) & 1023) - shift;
            const int valid = kFull ? 16 : (meta >> 20) & 31;
            // does the tile touch any row group of this wavefront?
            if (wi.n_grp == 0 || lo >= wi.n_grp || hi <= 0) return;
            Frag ks[4], vs[4];
            if (kFull || (!F8 && valid == 16)) {
                staged_operands(sb, ks, vs);
            } else {  // an open block: row-major in the stage buffer
#pragma unroll
                for (int r = 0; r < 4; ++r) ks[r].u = *reinterpret_cast<const u32x4*>(sb + c * 256 + g4 * 64 + r * 16);
                v_operands_from_rows(sb + 4096, 256, g4, c, vs);
            }
            // phase by phase over the row tiles, so that the products of one overlap the softmax of another
            f32x4 s[NT];
            bool on[NT], in_range[NT];
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) {
                on[nt] = NT == 1 || touches(nt, lo, hi);
                in_range[nt] = my_j[nt] >= lo && my_j[nt] < hi;
                if (on[nt]) s[nt] = products(ks, st[nt]);
            }
            if ((!kFull && valid < 16) || (meta >> 30)) {
#pragma unroll
                for (int nt = 0; nt < NT; ++nt)
                    if (on[nt]) mask_tokens(s[nt], visible(meta, my_j[nt] - lo), g4);
            }
            move_references<NT>(st, s, on, in_range, scale_log2e);
#pragma unroll
            for (int nt = 0; nt < NT; ++nt)
                if (on[nt]) weigh_values(vs, st[nt], s[nt], in_range[nt], scale_log2e);
        };
        // A full tile that every row group of the workgroup sees (the segments at the top of a unit: the common
        // case) needs no range, no mask and no decision per row tile: straight-line code around one rare branch
        // (the move of the references), a dozen scalar branches and a scalar load fewer per tile than the
        // general code.  Measured: 4 % off a prefill call, under 1 % off the decode calls.
        // Such tiles are taken in a loop of their own - inside one loop, next to the general code, the two
        // paths would disagree on the accumulators' registers and every tile would end in 64 register moves.
        auto consume_seen_by_all = [&](const char* sb) {
            if (wi.n_grp == 0) return;
            Frag ks[4], vs[4];
            staged_operands(sb, ks, vs);
            f32x4 s[NT];
            float top[NT];
            bool ran_away = false;
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) s[nt] = products(ks, st[nt]);
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) {
                top[nt] = top_logit(s[nt], my_j[nt] != 0x7fff, scale_log2e);
                ran_away = ran_away || top[nt] > st[nt].m + kSlack;
            }
            if (__builtin_amdgcn_ballot_w64(ran_away) != 0) {
#pragma unroll
                for (int nt = 0; nt < NT; ++nt) raise_reference(st[nt], top[nt]);
            }
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) weigh_values(vs, st[nt], s[nt], my_j[nt] != 0x7fff, scale_log2e);
        };
        // Two such tiles at once: twice as many independent chains of matrix instructions and one decision
        // about the references instead of two (a wavefront spends most of its time between dependent
        // instructions, not in them).
        auto consume_two_seen_by_all = [&](const char* sa, const char* sb) {
            if (wi.n_grp == 0) return;
            Frag ka[4], kb[4], va[4], vb[4];
#pragma unroll
            for (int r = 0; r < 4; ++r) ka[r].u = *reinterpret_cast<const u32x4*>(sa + r * 1024 + lane * 16);
#pragma unroll
            for (int r = 0; r < 4; ++r) kb[r].u = *reinterpret_cast<const u32x4*>(sb + r * 1024 + lane * 16);
#pragma unroll
            for (int r = 0; r < 4; ++r) va[r].u = *reinterpret_cast<const u32x4*>(sa + 4096 + r * 1024 + lane * 16);
#pragma unroll
            for (int r = 0; r < 4; ++r) vb[r].u = *reinterpret_cast<const u32x4*>(sb + 4096 + r * 1024 + lane * 16);
            f32x4 s0[NT], s1[NT];
            float top[NT];
            bool ran_away = false;
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) s0[nt] = products(ka, st[nt]);
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) s1[nt] = products(kb, st[nt]);
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) {
                const bool mine = my_j[nt] != 0x7fff;
                top[nt] = fmaxf(top_logit(s0[nt], mine, scale_log2e), top_logit(s1[nt], mine, scale_log2e));
                ran_away = ran_away || top[nt] > st[nt].m + kSlack;
            }
            if (__builtin_amdgcn_ballot_w64(ran_away) != 0) {
#pragma unroll
                for (int nt = 0; nt < NT; ++nt) raise_reference(st[nt], top[nt]);
            }
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) {
                weigh_values(va, st[nt], s0[nt], my_j[nt] != 0x7fff, scale_log2e);
                weigh_values(vb, st[nt], s1[nt], my_j[nt] != 0x7fff, scale_log2e);
            }
        };
        if (n_coop_full > 0) {  // the full tiles; which wavefront fetches is a scalar decision
            if (wave < n_coop_full) fetch_full(wave);
            // how many tiles at the head of the list are seen by all (the same count in every wavefront)
            int n_all = 0;
            for (int k = 0; k < 4; ++k)
                if (wg->w[k].n_grp > 0) n_all = max(n_all, wg->w[k].grp_lo + wg->w[k].n_grp - wg->grp_base);
            int n_lead = 0;
            for (int base = 0; base < n_coop_full; base += 64) {
                bool seen_by_all = false;
                if (base + lane < n_coop_full) {
                    const int meta = coop[base + lane].meta;
                    seen_by_all = (meta & 1023) == 0 && ((meta >> 10) & 1023) >= n_all && !(meta >> 30);
                }
                const uint64_t others = ~__builtin_amdgcn_ballot_w64(seen_by_all);
                const int run = others == 0 ? 64 : __builtin_ctzll(others);
                n_lead += run;
                if (run < 64) break;
            }
            // whole groups of four, or the whole list
            const int n_fast = n_lead >= n_coop_full ? n_coop_full : (n_lead & ~3);
            settle_queries();
            int t0 = 0;
            for (; t0 < n_fast; t0 += 4) {
                if (t0 > 0) __syncthreads();  // everyone is done reading the previous group
                if (t0 + wave < n_coop_full) to_stage(std::true_type{});
                __syncthreads();
                if (t0 + 4 + wave < n_coop_full) fetch_full(t0 + 4 + wave);
                const int n_here = min(4, n_coop_full - t0);
                int u = 0;
                for (; u + 1 < n_here; u += 2) consume_two_seen_by_all(stage[u], stage[u + 1]);
                if (u < n_here) consume_seen_by_all(stage[u]);
            }
            for (; t0 < n_coop_full; t0 += 4) {
                if (t0 > 0) __syncthreads();
                if (t0 + wave < n_coop_full) to_stage(std::true_type{});
                __syncthreads();
                if (t0 + 4 + wave < n_coop_full) fetch_full(t0 + 4 + wave);
                const int n_here = min(4, n_coop_full - t0);
                for (int u = 0; u < n_here; ++u) consume(t0 + u, stage[u], std::true_type{});
            }
        }
        if (n_coop_full < n_coop) {  // the open tiles
            if (n_coop_full > 0) __syncthreads();
            fetch_any(n_coop_full + wave);
            settle_queries();
            for (int t0 = n_coop_full; t0 < n_coop; t0 += 4) {
                if (t0 > n_coop_full) __syncthreads();
                if (t0 + wave < n_coop) to_stage(std::false_type{});
                __syncthreads();
                fetch_any(t0 + 4 + wave);
                const int n_here = min(4, n_coop - t0);
                for (int u = 0; u < n_here; ++u) consume(t0 + u, stage[u], std::false_type{});
            }
        }
        __syncthreads();  // the stage buffers are reused below
    }
    if (wi.n_grp == 0) return;  // a wavefront without rows only helped to fetch

    // ---- private tiles: straight into operand registers -------------------------------------
    // K pieces of a sealed tile are 1 KiB apart with the lanes side by side; of an open tile, 16 bytes
    // apart inside the lane's own 64 bytes of its token's row.  The V half is fetched raw either way.
    // K registers are refilled right after the K.Q^T products and V registers after the V^T.P^T products.
    Frag k[4], v[4];
    // fp8 pools: the codes of a full tile's halves as fetched, and the halves' scales; they become k, v just
    // before use (k_ready, v_ready), so that the codes of the next tile can be in flight meanwhile
    u32x4 k8[2], v8[2];
    float k8s = 1.0f, v8s = 1.0f;
    auto issue_k_full = [&](const char* tile) {
        const char* p = tile + lane * 16;
        if constexpr (F8) {
#pragma unroll
            for (int rp = 0; rp < 2; ++rp) k8[rp] = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(p + rp * 1024));
            k8s = scale_at(tile + kFp8ScaleOfs);
        } else {
#pragma unroll
            for (int r = 0; r < 4; ++r) k[r].u = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(p + r * 1024));
        }
    };
    auto issue_v_full = [&](const char* tile) {
        if constexpr (F8) {
            const char* p = tile + kFp8HalfBytes + lane * 16;
#pragma unroll
            for (int rp = 0; rp < 2; ++rp) v8[rp] = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(p + rp * 1024));
            v8s = scale_at(tile + kFp8ScaleOfs + 4);
        } else {
            const u32x4* p = reinterpret_cast<const u32x4*>(tile + 4096) + lane;
#pragma unroll
            for (int r = 0; r < 4; ++r) v[r].u = __builtin_nontemporal_load(p + r * 64);
        }
    };
    auto k_ready = [&](int valid) {  // (valid is wavefront-uniform)
        if constexpr (F8)
            if (valid == 16) fp8_operands(k8, k8s, k);
    };
    auto v_ready = [&](int valid) {
        if constexpr (F8)
            if (valid == 16) fp8_operands(v8, v8s, v);
    };
    // Only the filled rows of an open tile are read: a lane whose row lies past the fill count re-reads
    // row 0 (no branch around the loads, no extra traffic), and the masked logits give the slot probability 0.
    auto issue_k_open = [&](const char* tile, int valid) {
        const char* p = tile + (c < valid ? c : 0) * 256 + g4 * 64;
#pragma unroll
        for (int r = 0; r < 4; ++r) k[r].u = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(p + r * 16));
    };
    auto issue_v_open = [&](const char* tile, int valid) {
        const char* p = tile + 4096 + c * 16;
#pragma unroll
        for (int r = 0; r < 4; ++r) {  // raw piece r of this lane is part of token row 4r + g4
            const int row = 4 * r + g4 < valid ? 4 * r + g4 : 0;
            v[r].u = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(p + row * 256));
        }
    };
    char* scratch = lds + wave * kOpenScratch;
    const int n_full = own_full;
    int t = 0;
    int meta = 16 << 20;
    if (F8 && n_full > 2) {
        // fp8 pools: a tile is half the bytes, so one tile in flight per wavefront is half the bytes in flight,
        // too little to keep the memory system busy.  The full tiles but the last go through a pipeline two
        // tiles deep: two sets of raw registers, A (k8, v8) and B, tile j of the pipeline in one of them by
        // turns, each refilled with tile j + 2 as soon as its codes have been widened.  The last full tile L is
        // left in flight in set A for the loop below, as the one-deep loop leaves it.
        if constexpr (F8) {
            const int L = n_full - 1;
            u32x4 k8b[2], v8b[2];
            float k8sb = 1.0f, v8sb = 1.0f;
            auto load_raw = [&](const char* tile, u32x4 (&kk)[2], u32x4 (&vv)[2], float& ks, float& vs, bool want_k, bool want_v) {
                const char* p = tile + lane * 16;
                if (want_k) {
#pragma unroll
                    for (int rp = 0; rp < 2; ++rp) kk[rp] = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(p + rp * 1024));
                    ks = scale_at(tile + kFp8ScaleOfs);
                }
                if (want_v) {
#pragma unroll
                    for (int rp = 0; rp < 2; ++rp)
                        vv[rp] = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(p + kFp8HalfBytes + rp * 1024));
                    vs = scale_at(tile + kFp8ScaleOfs + 4);
                }
            };
            // tile j, whose codes are in (kk, vv); then (refill): tile j + 2 into the same registers
            auto step = [&](int j, u32x4 (&kk)[2], u32x4 (&vv)[2], float& ks, float& vs, bool refill) {
                const int mt = mine[j].meta;
                const int lo = mt & 1023, hi = (mt >> 10) & 1023;
                const char* tn = refill ? head_base + mine[j + 2].blk * block_stride : nullptr;
                f32x4 sj[NT];
                fp8_operands(kk, ks, k);
#pragma unroll
                for (int nt = 0; nt < NT; ++nt)
                    if (NT == 1 || touches(nt, lo, hi)) sj[nt] = products(k, st[nt]);
                if (refill) load_raw(tn, kk, vv, ks, vs, true, false);
                bool on[NT], in_range[NT];
#pragma unroll
                for (int nt = 0; nt < NT; ++nt) {
                    on[nt] = NT == 1 || touches(nt, lo, hi);
                    in_range[nt] = my_j[nt] >= lo && my_j[nt] < hi;
                    if (on[nt] && (mt >> 30)) mask_tokens(sj[nt], visible(mt, my_j[nt] - lo), g4);
                }
                move_references<NT>(st, sj, on, in_range, scale_log2e);
                fp8_operands(vv, vs, v);
#pragma unroll
                for (int nt = 0; nt < NT; ++nt)
                    if (on[nt]) weigh_values(v, st[nt], sj[nt], in_range[nt], scale_log2e);
                if (refill) load_raw(tn, kk, vv, ks, vs, false, true);
            };
            load_raw(head_base + mine[0].blk * block_stride, k8, v8, k8s, v8s, true, true);
            if (L & 1) {  // an odd number of tiles before the last: one of them alone, so that the rest go in pairs
                step(0, k8, v8, k8s, v8s, false);
                load_raw(head_base + mine[1].blk * block_stride, k8, v8, k8s, v8s, true, true);
                t = 1;
            }
            // L - t is even and at least 2: tiles t (in A) and t + 1 (into B) start the pairs
            load_raw(head_base + mine[t + 1].blk * block_stride, k8b, v8b, k8sb, v8sb, true, true);
            for (; t + 2 < L; t += 2) {
                step(t, k8, v8, k8s, v8s, true);
                step(t + 1, k8b, v8b, k8sb, v8sb, true);
            }
            step(t, k8, v8, k8s, v8s, true);          // refills A with tile L
            step(t + 1, k8b, v8b, k8sb, v8sb, false);
            t = L;
            meta = mine[L].meta;
        }
    } else if (n_full > 0) {
        // full tiles whose successor is full too: nothing but unconditional loads in this loop
        meta = mine[0].meta;
        const char* first = head_base + mine[0].blk * block_stride;
        issue_k_full(first);
        issue_v_full(first);
        for (; t + 1 < n_full; ++t) {
            const int lo = meta & 1023, hi = (meta >> 10) & 1023;
            const char* tn = head_base + mine[t + 1].blk * block_stride;
            const int meta_n = mine[t + 1].meta;
            f32x4 s[NT];
            k_ready(16);
#pragma unroll
            for (int nt = 0; nt < NT; ++nt)
                if (NT == 1 || touches(nt, lo, hi)) s[nt] = products(k, st[nt]);
            issue_k_full(tn);
            bool on[NT], in_range[NT];
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) {
                on[nt] = NT == 1 || touches(nt, lo, hi);
                in_range[nt] = my_j[nt] >= lo && my_j[nt] < hi;
                if (on[nt] && (meta >> 30)) mask_tokens(s[nt], visible(meta, my_j[nt] - lo), g4);
            }
            move_references<NT>(st, s, on, in_range, scale_log2e);
            v_ready(16);
#pragma unroll
            for (int nt = 0; nt < NT; ++nt)
                if (on[nt]) weigh_values(v, st[nt], s[nt], in_range[nt], scale_log2e);
            issue_v_full(tn);
            meta = meta_n;
        }
    } else if (wi.n_tiles > 0) {
        meta = mine[0].meta;
        const char* first = head_base + mine[0].blk * block_stride;
        issue_k_open(first, (meta >> 20) & 31);
        issue_v_open(first, (meta >> 20) & 31);
    }
    // The last full tile and the open tiles.  Every successor is open, so the loads of this loop are unconditional too and none
    // lies behind a branch on the tile at hand; after the last tile one row of it is fetched again and not looked at.  With the
    // V half turned by transposing LDS reads (thirty-two 2-byte reads per lane before) and the loads out of the branches: one
    // request of five threads 13.5 -> 12.8 us, 256 requests on an fp8 pool 1014 -> 994, five candidates 1008 -> 998.
    auto last_tile_or_open = [&](auto maybe_full, const char* tn, int valid_n) {
        const int lo = meta & 1023, hi = (meta >> 10) & 1023;
        const int valid = F8 ? (decltype(maybe_full)::value ? 16 : min(15, (meta >> 20) & 31)) : (meta >> 20) & 31;
        f32x4 s[NT];
        k_ready(valid);
#pragma unroll
        for (int nt = 0; nt < NT; ++nt)
            if (NT == 1 || touches(nt, lo, hi)) s[nt] = products(k, st[nt]);
        issue_k_open(tn, valid_n);  // K registers are free again
        if (valid < 16) {
            // open block: its V half arrived row-major; turn it into operand order through LDS
#pragma unroll
            for (int r = 0; r < 4; ++r)
                *reinterpret_cast<u32x4*>(scratch + (4 * r + g4) * kOpenRowStride + c * 16) = v[r].u;
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
            v_operands_from_rows(scratch, kOpenRowStride, g4, c, v);
            __builtin_amdgcn_wave_barrier();
        }
        v_ready(valid);
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
            if (NT > 1 && !touches(nt, lo, hi)) continue;
            if (valid < 16 || (meta >> 30)) mask_tokens(s[nt], visible(meta, my_j[nt] - lo), g4);
            accumulate(v, st[nt], s[nt], my_j[nt] >= lo && my_j[nt] < hi, scale_log2e);
        }
        issue_v_open(tn, valid_n);
    };
    auto go_on = [&](auto maybe_full) {
        const bool more = t + 1 < wi.n_tiles;
        const TileRef next = mine[more ? t + 1 : t];
        last_tile_or_open(maybe_full, head_base + next.blk * block_stride, more ? (next.meta >> 20) & 31 : 1);
        meta = next.meta;
        ++t;
    };
    if (F8 && n_full > 0) go_on(std::true_type{});
    while (t < wi.n_tiles) go_on(std::false_type{});

    // ---- results ------------------------------------------------------------------------------
    if (NT == 1 && (wi.flags & kWaveSplit)) {
        // the four wavefronts hold the same rows over different tiles: fold 1..3 into 0 through LDS, every register of a
        // wavefront as 1 KiB in the order of its lanes (row by row instead, sixteen lanes met in one bank: one request of five
        // threads, 32 heads 15.5 us per call instead of 14.9)
        RowState& s0 = st[0];
        __syncthreads();  // every wavefront is done with its transpose scratch, which this area overlaps
        if (wave > 0) {
            char* to = lds + (wave - 1) * kSplitState;
#pragma unroll
            for (int jj = 0; jj < 8; ++jj) *reinterpret_cast<f32x4*>(to + (jj * 64 + lane) * 16) = s0.o[jj];
            *reinterpret_cast<f32x2*>(to + 8 * 1024 + lane * 8) = f32x2{s0.m, s0.l};
        }
        __syncthreads();
        if (wave > 0) return;
        f32x2 ml[3];
        float mx = s0.m;
#pragma unroll
        for (int w2 = 0; w2 < 3; ++w2) {
            ml[w2] = *reinterpret_cast<const f32x2*>(lds + w2 * kSplitState + 8 * 1024 + lane * 8);
            mx = fmaxf(mx, ml[w2].x);
        }
        // a wavefront that saw no tile of a row left m = -inf and sums of zero for it
        const float a0 = (s0.m == -INFINITY) ? 0.0f : __builtin_amdgcn_exp2f(s0.m - mx);
        s0.l *= a0;
#pragma unroll
        for (int jj = 0; jj < 8; ++jj) s0.o[jj] *= a0;
#pragma unroll
        for (int w2 = 0; w2 < 3; ++w2) {
            const float aw = (ml[w2].x == -INFINITY) ? 0.0f : __builtin_amdgcn_exp2f(ml[w2].x - mx);
            s0.l += aw * ml[w2].y;
#pragma unroll
            for (int jj = 0; jj < 8; ++jj)
                s0.o[jj] += aw * *reinterpret_cast<const f32x4*>(lds + w2 * kSplitState + (jj * 64 + lane) * 16);
        }
        s0.m = mx;
        __builtin_amdgcn_wave_barrier();
    }

    if ((wi.flags & kWaveDirect) && cand_mask != nullptr && (!SPLIT || slice.s == 0))
        attend_candidates<NT>(st, scratch, plan, wi, cand_k, cand_v, cand_mask, my_j, within, n_cand, n_kv, kvh, group, scale_log2e);

    if constexpr (SPLIT)
        if (!fold_slices<NT, 8>(plan.split, slice, n_kv, kvh, wave, (wi.flags & kWaveSplit) ? 1 : 4, lane, st)) return;

#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
        float lt = st[nt].l;
        lt += __shfl_xor(lt, 16, 64);
        lt += __shfl_xor(lt, 32, 64);
        int rk = 0, r2 = 0;
        int64_t qrow = -1, slot = 0;
        if (my_j[nt] != 0x7fff) locate(nt, rk, r2, qrow, slot);
        if (wi.flags & kWaveDirect) {
            // The row's whole root path was covered here: normalise and write the output row - through LDS, so that a
            // store instruction writes four whole rows of 256 bytes (a lane holds its row in runs of four dims).  Against
            // stores of 8 bytes per lane: 15 k threads, 8 kv heads 3184 -> 3141 us, 3.8 k threads, 32 kv heads 1503 -> 1489;
            // with plain instead of non-temporal stores the latter takes 1527.
            const float inv = 1.0f / lt;
            __builtin_amdgcn_wave_barrier();
#pragma unroll
            for (int jj = 0; jj < 8; ++jj) {
                u32x2 pk;
                pk.x = pack_bf16_pair(st[nt].o[jj][0] * inv, st[nt].o[jj][1] * inv);
                pk.y = pack_bf16_pair(st[nt].o[jj][2] * inv, st[nt].o[jj][3] * inv);
                *reinterpret_cast<u32x2*>(scratch + c * kOpenRowStride + 32 * jj + 8 * g4) = pk;
            }
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll
            for (int it = 0; it < 4; ++it) {
                const int r = 4 * it + g4;  // (lane r knows where row r goes)
                const int64_t row = __shfl((long long)qrow, r, 64);
                const u32x4 x = *reinterpret_cast<const u32x4*>(scratch + r * kOpenRowStride + c * 16);
                if (row >= 0) __builtin_nontemporal_store(x, reinterpret_cast<u32x4*>(out + row * 128) + c);
            }
        } else if (my_j[nt] != 0x7fff) {
            float* dst = part.o + slot * 128 + 4 * g4;
            if (part.stream) {
                asm volatile("" ::: "memory");  // (before and after: else the two branches' stores become one, without the hint)
#pragma unroll
                for (int jj = 0; jj < 8; ++jj) __builtin_nontemporal_store(st[nt].o[jj], reinterpret_cast<f32x4*>(dst + 16 * jj));
                asm volatile("" ::: "memory");
            } else {  // 64 bytes per row and store, which the L2 puts together, and the merge kernel finds them there
#pragma unroll
                for (int jj = 0; jj < 8; ++jj) *reinterpret_cast<f32x4*>(dst + 16 * jj) = st[nt].o[jj];
            }
            if (g4 == 0) {
                part.ml[slot * 2] = st[nt].m;
                part.ml[slot * 2 + 1] = lt;
            }
        }
    }
}

// Units of one row-tile class.  INLINE (with SPLIT): the plan's tables come with the kernel's arguments.
template <int NT, bool F8, bool SPLIT, bool INLINE>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(NT == 1 ? 3 : 2))) void attention_bf16(
    PlanWords<INLINE>, const char* __restrict__ pool, const uint16_t* __restrict__ q, PlanDev plan, int wg_first, int n_cand, int n_q, int n_kv,
    int group, float scale_log2e, PartialBuf part, const uint16_t* __restrict__ cand_k, const uint16_t* __restrict__ cand_v,
    const uint8_t* __restrict__ cand_mask, uint16_t* __restrict__ out) {
    __shared__ __attribute__((aligned(16))) char lds[kAttnLds];
    const Slice slice = unit_of_block<SPLIT, INLINE>(plan, wg_first, n_kv);
    attend_unit<NT, F8, SPLIT>(lds, slice, pool, q, plan, n_cand, n_q, n_kv, group, scale_log2e, part, cand_k, cand_v, cand_mask, out);
}

// Units of both classes in one launch (217 to 240 registers: the chip holds two workgroups per compute unit, where units of one
// row tile alone would have three).  Two launches side by side cost an event, two waits and the second stream's start, and each
// ends on a tail of its own.  Measured, us per call, two launches / one (workgroups of the two classes):
//   bf16   8 kv heads (16 + 1016) 176 / 134, (96 + 4032) 564 / 475, (48 + 8160) 979 / 888, (792 + 3600) 711 / 664, 84 requests of two
//          fork levels 207 / 168, 128 requests of group 8 246 / 211, 1024 of group 4 3136 / 3060; 32 kv heads (32 + 2016) 301 / 226,
//          (32 + 8160) 810 / 645, (832 + 7360) 1854 / 1753; two candidates (64 requests) 583 / 441, three 502 / 469, (100) 339 / 339;
//          five (2368 + 2112) 915 / 868, (9536 + 576) 3278 / 3261, (29408 + 192) 11680 / 11720
//   fp8    8 kv heads (16 + 1016) 127 / 80, (96 + 4032) 342 / 262, (48 + 8160) 557 / 489, (792 + 3600) 460 / 413; 32 kv heads (32 + 2016)
//          232 / 166, (32 + 8160) 487 / 367, (832 + 7360) 1461 / 1340; two candidates (224 + 3968) 276 / 199
template <bool F8, bool SPLIT, bool INLINE>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2))) void attention_bf16_both(
    PlanWords<INLINE>, const char* __restrict__ pool, const uint16_t* __restrict__ q, PlanDev plan, int wg_first, int n_cand, int n_q, int n_kv,
    int group, float scale_log2e, PartialBuf part, const uint16_t* __restrict__ cand_k, const uint16_t* __restrict__ cand_v,
    const uint8_t* __restrict__ cand_mask, uint16_t* __restrict__ out) {
    __shared__ __attribute__((aligned(16))) char lds[kAttnLds];
    const Slice slice = unit_of_block<SPLIT, INLINE>(plan, wg_first, n_kv);
    tables_unwritten(plan);
    if ((plan.wgs[slice.wg].row_tiles & 255) == 2)
        attend_unit<2, F8, SPLIT>(lds, slice, pool, q, plan, n_cand, n_q, n_kv, group, scale_log2e, part, cand_k, cand_v, cand_mask, out);
    else
        attend_unit<1, F8, SPLIT>(lds, slice, pool, q, plan, n_cand, n_q, n_kv, group, scale_log2e, part, cand_k, cand_v, cand_mask, out);
}

}  // namespace

hipError_t launch_attention_bf16(const Shape& s, const void* pool, const void* q, const PlanDev& plan, int n_cand,
                                 PartialBuf part, const void* cand_k, const void* cand_v, const uint8_t* mask,
                                 void* out, hipStream_t st) {
    // workgroups are sorted by class: [matrix units | 2 row tiles per wavefront | 1], heaviest first in each.
    // Matrix units go first, alone: their workgroups need 64 KB of LDS and most of a
    // SIMD's registers, and beside a kernel of small workgroups they wait until that kernel has drained
    // (measured: a 100 us launch took as long as the 800 us launch beside it).
    if (plan.few != 2 && plan.n_inline_words > kPlanInlineWords) return hipErrorInvalidValue;
    const bool split = plan.split.blocks != nullptr || plan.inline_words;
    const int32_t* n_class = split ? plan.split.n_blocks_class : plan.n_wg_class;  // (matrix units are never cut)
    const int first = n_class[0];
    const int64_t n_wg = ((int64_t)n_class[1] + n_class[2]) * s.n_kv;
    if (n_wg > 0x7fffffff) return hipErrorInvalidValue;
    hipError_t e;
    if (first > 0 && (e = launch_attention_units_bf16(s, pool, q, plan, 0, first, n_cand, part, st)) != hipSuccess) return e;
    if (n_wg == 0) return hipSuccess;
    if (plan.few) return launch_attention_few_bf16(s, pool, q, plan, n_cand, part, cand_k, cand_v, mask, out, st);
#define APAR_LAUNCH(KERNEL, WORDS)                                                                                      \
    hipLaunchKernelGGL(KERNEL, dim3((unsigned)n_wg), dim3(256), 0, st, WORDS,                                            \
                       (const char*)pool, (const uint16_t*)q, plan, first, n_cand, s.n_q, s.n_kv, s.group,               \
                       s.scale_log2e, part, (const uint16_t*)cand_k, (const uint16_t*)cand_v, mask, (uint16_t*)out)
#define APAR_LAUNCH_CLASS(F8V, SPLITV, INLINEV, WORDS)                                                  \
    do {                                                                                                \
        if (n_class[1] == 0) APAR_LAUNCH((attention_bf16<1, F8V, SPLITV, INLINEV>), WORDS);             \
        else if (n_class[2] == 0) APAR_LAUNCH((attention_bf16<2, F8V, SPLITV, INLINEV>), WORDS);        \
        else APAR_LAUNCH((attention_bf16_both<F8V, SPLITV, INLINEV>), WORDS);                           \
    } while (0)
#define APAR_LAUNCH_F8(SPLITV, INLINEV, WORDS)                              \
    do {                                                                    \
        if (s.fp8_sealed) APAR_LAUNCH_CLASS(true, SPLITV, INLINEV, WORDS);  \
        else APAR_LAUNCH_CLASS(false, SPLITV, INLINEV, WORDS);              \
    } while (0)
    if (plan.inline_words) {
        PlanWords<true> words;
        memcpy(words.words, plan.inline_words, (size_t)plan.n_inline_words * sizeof(int32_t));
        APAR_LAUNCH_F8(true, true, words);
    } else if (split) {
        APAR_LAUNCH_F8(true, false, PlanWords<false>{});
    } else {
        APAR_LAUNCH_F8(false, false, PlanWords<false>{});
    }
#undef APAR_LAUNCH_F8
#undef APAR_LAUNCH_CLASS
#undef APAR_LAUNCH
    return hipGetLastError();
}

}  // namespace apar
