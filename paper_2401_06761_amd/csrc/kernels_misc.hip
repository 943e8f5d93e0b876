// Row writes, copy-on-write block copies, row read-back and the merge kernel (gfx950).
#include <hip/hip_runtime.h>

#include <cstring>

#include "apar_internal.hpp"

namespace apar {

namespace {

__device__ __forceinline__ float bf16_to_f32(uint16_t b) { return __uint_as_float((uint32_t)b << 16); }

__device__ __forceinline__ uint16_t f32_to_bf16_rne(float f) {
    uint32_t u = __float_as_uint(f);
    if ((u & 0x7fffffffu) > 0x7f800000u) return (uint16_t)((u >> 16) | 0x40);  // quiet NaN
    u += 0x7fffu + ((u >> 16) & 1u);
    return (uint16_t)(u >> 16);
}

// ---------------------------------------------------------------------------
// Appended rows, one pass per block: a wavefront takes one (block the call writes to, kv head).  The block's rows
// [s0, s1) come from the call's k and v; where the block is the copy-on-write copy of a shared tail, rows [0, s0) come
// from that.  A block that stays open is written row by row (256 or 512 contiguous bytes a half).  A block that is full
// now (16-bit pools) is SEALED: its sixteen rows are gathered in LDS - those before s0 from the block itself or from the
// block it copies - and written once, in matrix-core order.
// Before, three kernels did this: block copies, row writes, and a pass that read full blocks back and rewrote them.
// Their time against this kernel's (us, with the two events around them): prompts of 300, 1 k, 4 k, 8 k rows, 8 kv heads
// 8.9, 10.0, 17.5, 28.3 -> 6.8, 7.8, 9.6, 14.2; one row each for 3.8 k threads, 32 heads, one in sixteen sealing 56 -> 47;
// 5 and 1000 threads forked off a tail of 9 rows 11.2, 74 -> 8.7, 45, off one of 15 (copied and sealed) 10.8, 194 -> 6.9, 67.
// ---------------------------------------------------------------------------
// A tile half's rows in LDS: padded, so that sixteen lanes reading one piece of sixteen rows meet sixteen banks.
constexpr int kSealRowStride = 272;
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

// fp8 pools: the smallest power of two s for which max |x| / s <= 448, the largest e4m3 magnitude (1 if the half is
// all zeros), so that the codes use the top binade of the format.  Codes are rounded to nearest even by the hardware
// conversion.
__device__ __forceinline__ float fp8_scale_for(float amax) {
    if (!(amax > 0.0f) || !(amax < INFINITY)) return 1.0f;
    int k;
    const float f = frexpf(amax, &k);            // amax = f * 2^k, f in [0.5, 1); 448 = 0.875 * 2^9
    const int e = (f <= 0.875f) ? k - 9 : k - 8;
    return ldexpf(1.0f, e < -126 ? -126 : e);
}

// One half of a tile, its sixteen rows in LDS, in matrix-core order (a lane's pieces r = 0..3; see the pool layout):
// K[token c][dims 32g + 8r .. +8];  V[tokens 4g..4g+3][dim 32r + c], then [dim 32r + 16 + c].
__device__ __forceinline__ void k_piece(const char* rows, int lane, int r, uint16_t (&x)[8]) {
    *reinterpret_cast<uint4*>(x) = *reinterpret_cast<const uint4*>(rows + (lane & 15) * kSealRowStride + (32 * (lane >> 4) + 8 * r) * 2);
}
__device__ __forceinline__ void v_piece(const char* rows, int lane, int r, uint16_t (&x)[8]) {
#pragma unroll
    for (int hh = 0; hh < 2; ++hh)
#pragma unroll
        for (int i = 0; i < 4; ++i)
            x[4 * hh + i] = *reinterpret_cast<const uint16_t*>(rows + (4 * (lane >> 4) + i) * kSealRowStride + (32 * r + 16 * hh + (lane & 15)) * 2);
}

// fp8 codes of a piece under the inverse of the half's scale (a power of two: exact)
__device__ __forceinline__ uint2 fp8_piece(const uint16_t (&x)[8], float inv) {
    uint32_t w[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        w[i] = __builtin_amdgcn_cvt_pk_fp8_f32(bf16_to_f32(x[4 * i]) * inv, bf16_to_f32(x[4 * i + 1]) * inv, 0, false);
        w[i] = __builtin_amdgcn_cvt_pk_fp8_f32(bf16_to_f32(x[4 * i + 2]) * inv, bf16_to_f32(x[4 * i + 3]) * inv, w[i], true);
    }
    return make_uint2(w[0], w[1]);
}

// ROW: bytes of one row of a half.  SEAL: 0 fp32 pools (nothing is sealed), 1 bf16, 2 fp8.  FROM: where the descriptors and
// the source rows are (in the kernel's arguments: its first one, so that they start the argument segment).  Blocks of a run go along
// with a word each: a prompt of 2 k to 8 k tokens (8 kv heads) does without the copy of its table and the gap behind it (six such prompts
// and their attention 1763 -> 1720 us).
// In the tables the blocks that stay open come first, n_open of them.  The first workgroups take the full ones, a wavefront per
// (block, kv head), so that the launch does not end on them; the others write the open ones, as many lanes as a row has
// 16-byte pieces per (block, kv head).  A full block's earlier rows are read with non-temporal loads, other rows (the caller's,
// shared tails) with plain ones.  Measured, us: 3.8 k threads, 32 heads, one row each, one block in sixteen full: full blocks
// last 59.6, first 56.4, non-temporal loads for their own rows 47.0; for every row 51.4, and 1000 copies of a tail of 9
// rows 76 instead of 44.
template <int ROW, int SEAL, int FROM>
__global__ __launch_bounds__(256) void append_blocks(AppendTables<FROM> tables, char* __restrict__ pool, const char* __restrict__ k,
                                                     const char* __restrict__ v, int n_blocks, int n_open, int n_src, int n_kv) {
    // one half's rows per wavefront: the open blocks' workgroups want the occupancy
    __shared__ __attribute__((aligned(16))) char lds[SEAL ? 4 : 1][SEAL ? 16 * kSealRowStride : 16];
    constexpr int64_t kTile = 2 * 16 * ROW;
    constexpr int kLanes = 2 * ROW / 16;      // lanes of one row: its K half, then its V half
    auto block_at = [&](int at) -> AppendBlock {
        if constexpr (FROM == kAppendRun) {
            typedef const int32_t __attribute__((address_space(4))) * Words;
            const auto w = (Words)__builtin_amdgcn_kernarg_segment_ptr();
            const int before = w[0];
            if (at < before) return AppendBlock{w[4 + 4 * at], w[5 + 4 * at], w[6 + 4 * at], w[7 + 4 * at]};
            return AppendBlock{w[4 + 3 * before + at], -1, w[1] + 16 * (at - before), 16 << 8};
        } else if constexpr (FROM == kAppendArguments) {
            typedef const AppendBlock __attribute__((address_space(4))) * Blocks;
            const auto* p = (Blocks)__builtin_amdgcn_kernarg_segment_ptr() + at;
            return AppendBlock{p->dst, p->copy_of, p->first, p->slots};
        } else {
            return reinterpret_cast<const AppendBlock*>(tables.words)[at];
        }
    };
    auto src_of = [&](int i) -> int {
        if constexpr (FROM == kAppendRun) {
            return i;  // (a run has no list of source rows)
        } else if constexpr (FROM == kAppendArguments) {
            typedef const int32_t __attribute__((address_space(4))) * Words;
            return ((Words)__builtin_amdgcn_kernarg_segment_ptr())[4 * n_blocks + i];
        } else {
            return tables.words[4 * n_blocks + i];
        }
    };
    // where 16 bytes of slot `slot` (before s1) of a block come from, at `ofs` of half `half` (one load, whose address is
    // chosen: a branch around it would make every load wait where it is issued)
    auto source = [&](const AppendBlock& b, int h, int half, int slot, int ofs) -> const u32x4* {
        const int s0 = b.slots & 255, row = b.first + max(slot - s0, 0);
        const int64_t from = n_src ? src_of(row) : row;
        const char* fresh = (half ? v : k) + (from * n_kv + h) * ROW;
        const char* old = pool + ((int64_t)(b.copy_of >= 0 ? b.copy_of : b.dst) * n_kv + h) * kTile + half * 16 * ROW + slot * ROW;
        return reinterpret_cast<const u32x4*>((slot < s0 ? old : fresh) + ofs);
    };
    constexpr int kPairs = 256 / kLanes;
    const int full_wgs = SEAL ? (int)(((int64_t)(n_blocks - n_open) * n_kv + 3) / 4) : 0;
    if ((int)blockIdx.x >= full_wgs) {
        const int pair = ((int)blockIdx.x - full_wgs) * kPairs + (int)threadIdx.x / kLanes;  // (open block, kv head), heads fastest
        const int at = pair / n_kv, h = pair - at * n_kv;
        if (at >= n_open) return;
        const AppendBlock b = block_at(at);
        const int l = (int)threadIdx.x % kLanes, half = l / (kLanes / 2), ofs = (l % (kLanes / 2)) * 16;
        char* dst = pool + ((int64_t)b.dst * n_kv + h) * kTile + half * 16 * ROW + ofs;
        const int s1 = b.slots >> 8;
        int s = b.copy_of >= 0 ? 0 : b.slots & 255;
        if (s + 1 == s1) {
            *reinterpret_cast<u32x4*>(dst + s * ROW) = *source(b, h, half, s, ofs);
            return;
        }
        for (; s < s1; s += 4) {  // four rows in flight
            u32x4 x[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) x[i] = *source(b, h, half, min(s + i, s1 - 1), ofs);
#pragma unroll
            for (int i = 0; i < 4; ++i)
                if (s + i < s1) *reinterpret_cast<u32x4*>(dst + (s + i) * ROW) = x[i];
        }
        return;
    }
    if constexpr (SEAL != 0) {
        const int lane = threadIdx.x & 63;
        const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
        const int item = (int)blockIdx.x * 4 + wave;  // (full block, kv head), heads fastest
        const int at = item / n_kv, h = item - at * n_kv;
        if (at >= n_blocks - n_open) return;
        const AppendBlock b = block_at(n_open + at);
        constexpr int kRows = 64 / kLanes;    // rows a wavefront moves at once
        const int l = lane % kLanes, half = l / (kLanes / 2), chunk = (l % (kLanes / 2)) * 16, sub = lane / kLanes;
        char* tile = pool + ((int64_t)b.dst * n_kv + h) * kTile;
        char* rows = lds[wave];
        u32x4 x[16 / kRows];
        if (b.copy_of < 0 && (b.slots & 255) > 0) {  // its own rows so far, laid out anew: not read again as they are
#pragma unroll
            for (int i = 0; i < 16 / kRows; ++i) x[i] = __builtin_nontemporal_load(source(b, h, half, i * kRows + sub, chunk));
        } else {
#pragma unroll
            for (int i = 0; i < 16 / kRows; ++i) x[i] = *source(b, h, half, i * kRows + sub, chunk);
        }
        float scale[2] = {1.0f, 1.0f};
        if constexpr (SEAL == 2) {
            float top = 0.0f;
#pragma unroll
            for (int i = 0; i < 16 / kRows; ++i) {
                const uint32_t w[4] = {x[i].x, x[i].y, x[i].z, x[i].w};
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    top = fmaxf(top, fmaxf(fabsf(__uint_as_float(w[e] << 16)), fabsf(__uint_as_float(w[e] & 0xffff0000u))));
            }
#pragma unroll
            for (int o = 1; o < 64; o <<= 1)
                if (o != kLanes / 2) top = fmaxf(top, __shfl_xor(top, o, 64));
            const float other = __shfl_xor(top, kLanes / 2, 64);
            scale[0] = fp8_scale_for(half ? other : top);
            scale[1] = fp8_scale_for(half ? top : other);
        }
        // (every row is in registers by the time the first piece is written: the tile may be overwritten in place)
#pragma unroll
        for (int hf = 0; hf < 2; ++hf) {
            __builtin_amdgcn_wave_barrier();
            if (half == hf) {
#pragma unroll
                for (int i = 0; i < 16 / kRows; ++i) *reinterpret_cast<u32x4*>(rows + (i * kRows + sub) * kSealRowStride + chunk) = x[i];
            }
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                __attribute__((aligned(16))) uint16_t e[8];
                if (hf == 0) k_piece(rows, lane, r, e);
                else v_piece(rows, lane, r, e);
                if constexpr (SEAL == 2)
                    *reinterpret_cast<uint2*>(tile + hf * kFp8HalfBytes + (r >> 1) * 1024 + lane * 16 + (r & 1) * 8) = fp8_piece(e, 1.0f / scale[hf]);
                else
                    *reinterpret_cast<uint4*>(tile + hf * 4096 + r * 1024 + lane * 16) = *reinterpret_cast<const uint4*>(e);
            }
        }
        if constexpr (SEAL == 2)
            if (lane == 0) *reinterpret_cast<float2*>(tile + kFp8ScaleOfs) = make_float2(scale[0], scale[1]);
    }
}

__global__ __launch_bounds__(64) void read_rows_bf16(const char* __restrict__ pool, uint16_t* __restrict__ k,
                                                     uint16_t* __restrict__ v, const int32_t* __restrict__ codes,
                                                     int n_kv, int64_t tile_bytes, int fp8_sealed) {
    const int row = blockIdx.x, h = blockIdx.y, lane = threadIdx.x;
    const int32_t code = codes[row];
    const bool sealed = (code & kCodeSealed) != 0;  // the row's block is full, hence in matrix-core order
    const int slot = code & 15;
    const char* tile = pool + ((int64_t)((code & ~kCodeSealed) >> 4) * n_kv + h) * tile_bytes;
    uint16_t* kdst = k + ((int64_t)row * n_kv + h) * 128;
    uint16_t* vdst = v + ((int64_t)row * n_kv + h) * 128;
    if (sealed && fp8_sealed) {  // fp8 codes times the half's power-of-two scale: exact in bf16
        const float2 sc = *reinterpret_cast<const float2*>(tile + kFp8ScaleOfs);
#pragma unroll
        for (int e = 0; e < 2; ++e) {
            const int dim = lane + 64 * e;
            const uint32_t kc = *reinterpret_cast<const uint8_t*>(tile + fp8_k_offset(slot, dim));
            const uint32_t vc = *reinterpret_cast<const uint8_t*>(tile + kFp8HalfBytes + fp8_v_offset(slot, dim));
            kdst[dim] = f32_to_bf16_rne(__builtin_amdgcn_cvt_f32_fp8(kc, 0) * sc.x);
            vdst[dim] = f32_to_bf16_rne(__builtin_amdgcn_cvt_f32_fp8(vc, 0) * sc.y);
        }
        return;
    }
#pragma unroll
    for (int e = 0; e < 2; ++e) {
        const int dim = lane + 64 * e;
        const int ko = sealed ? bf16_k_offset(slot, dim) : slot * 256 + dim * 2;
        const int vo = sealed ? bf16_v_offset(slot, dim) : slot * 256 + dim * 2;
        kdst[dim] = *reinterpret_cast<const uint16_t*>(tile + ko);
        vdst[dim] = *reinterpret_cast<const uint16_t*>(tile + 4096 + vo);
    }
}

__global__ __launch_bounds__(64) void read_rows_f32(const char* __restrict__ pool, float* __restrict__ k,
                                                    float* __restrict__ v, const int32_t* __restrict__ codes,
                                                    int n_kv, int d, int64_t tile_bytes) {
    const int row = blockIdx.x, h = blockIdx.y, lane = threadIdx.x;
    const int32_t code = codes[row];
    const int slot = code & 15;
    const float* tile = reinterpret_cast<const float*>(pool + ((int64_t)(code >> 4) * n_kv + h) * tile_bytes);
    for (int x = lane; x < d; x += 64) {
        k[((int64_t)row * n_kv + h) * d + x] = tile[slot * d + x];
        v[((int64_t)row * n_kv + h) * d + x] = tile[16 * d + slot * d + x];
    }
}

// Copy-on-write: whole blocks, 16 bytes per lane.  grid = (pairs, slices).
__global__ __launch_bounds__(256) void copy_blocks(char* __restrict__ pool, const int32_t* __restrict__ pairs,
                                                   int64_t block_bytes) {
    const int32_t src = pairs[2 * blockIdx.x], dst = pairs[2 * blockIdx.x + 1];
    const uint4* s = reinterpret_cast<const uint4*>(pool + (int64_t)src * block_bytes);
    uint4* d = reinterpret_cast<uint4*>(pool + (int64_t)dst * block_bytes);
    const int64_t n16 = block_bytes / 16;
    for (int64_t i = (int64_t)blockIdx.y * blockDim.x + threadIdx.x; i < n16; i += (int64_t)gridDim.y * blockDim.x)
        d[i] = s[i];
}

// ---------------------------------------------------------------------------
// Merge: sixteen lanes per (listed thread, candidate, q head).  Folds the partial
// results on the thread's root path (log-sum-exp in base 2), adds the candidate
// keys the mask lets this candidate see, normalises and writes the output row.
// Threads without partial results were already written by the attention kernel.
// ---------------------------------------------------------------------------
// E consecutive elements starting at element idx (a multiple of E) as floats: 16-byte loads.
template <int E, bool BF16>
__device__ __forceinline__ void load_run(const void* base, int64_t idx, float (&x)[E]) {
    if constexpr (BF16) {
        static_assert(E == 8, "a bf16 run is one 16-byte load");
        const uint4 u = *reinterpret_cast<const uint4*>(reinterpret_cast<const uint16_t*>(base) + idx);
        const uint32_t w[4] = {u.x, u.y, u.z, u.w};
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            x[2 * e] = __uint_as_float(w[e] << 16);
            x[2 * e + 1] = __uint_as_float(w[e] & 0xffff0000u);
        }
    } else {
#pragma unroll
        for (int e = 0; e < E; e += 4) {
            const float4 f = *reinterpret_cast<const float4*>(reinterpret_cast<const float*>(base) + idx + e);
            x[e] = f.x, x[e + 1] = f.y, x[e + 2] = f.z, x[e + 3] = f.w;
        }
    }
}

__device__ __forceinline__ float sum_over_16_lanes(float x) {
#pragma unroll
    for (int o = 8; o > 0; o >>= 1) x += __shfl_xor(x, o, 64);
    return x;
}

// A workgroup takes 16 consecutive q heads of one (listed thread, candidate): sixteen lanes per output
// row, each with D / 16 consecutive dims, so the four rows of a wavefront read 4 * D consecutive floats
// of every partial result in one go.
template <int D, bool BF16>
__global__ __launch_bounds__(256) void merge_rows(PlanDev plan, PartialBuf part, const void* __restrict__ qv,
                                                  const void* __restrict__ ckv, const void* __restrict__ cvv,
                                                  const uint8_t* __restrict__ mask, int n_cand, int n_q, int n_kv,
                                                  int group, float scale_log2e, void* __restrict__ outv) {
    constexpr int E = D / 16;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int c16 = lane & 15;
    const int head = blockIdx.x * 16 + wave * 4 + (lane >> 4);
    const int c = blockIdx.y, i = blockIdx.z;
    const int p0 = plan.path_ofs[i], p1 = plan.path_ofs[i + 1];
    if (p0 == p1) return;  // the attention kernel wrote this thread's rows itself (candidates included)
    const bool ok = head < n_q;
    const int hq = ok ? head : 0;  // rows past the last head redo head 0 and write nothing
    float m = -INFINITY;
    for (int p = p0; p < p1; ++p) {
        const int64_t slot = ((int64_t)plan.path_ids[p] * n_cand + c) * n_q + hq;
        m = fmaxf(m, part.ml[slot * 2]);
    }
    // logits of the visible candidates
    float cs[8];
    uint32_t bits = 0;
    if (mask != nullptr) {
        bits = mask[(int64_t)i * n_cand + c];
        float qr[E];
        load_run<E, BF16>(qv, (((int64_t)i * n_cand + c) * n_q + hq) * D + c16 * E, qr);
        for (int cp = 0; cp < n_cand; ++cp) {
            cs[cp] = -INFINITY;
            if ((bits >> cp) & 1u) {
                float kr[E];
                load_run<E, BF16>(ckv, (((int64_t)i * n_cand + cp) * n_kv + hq / group) * D + c16 * E, kr);
                float dot = 0.0f;
#pragma unroll
                for (int e = 0; e < E; ++e) dot += qr[e] * kr[e];
                cs[cp] = sum_over_16_lanes(dot) * scale_log2e;
                m = fmaxf(m, cs[cp]);
            }
        }
    }
    float l = 0.0f, acc[E];
#pragma unroll
    for (int e = 0; e < E; ++e) acc[e] = 0.0f;
#pragma unroll 2
    for (int p = p0; p < p1; ++p) {
        const int64_t slot = ((int64_t)plan.path_ids[p] * n_cand + c) * n_q + hq;
        const float2 ml = *reinterpret_cast<const float2*>(part.ml + slot * 2);
        float o[E];
        load_run<E, false>(part.o, slot * D + c16 * E, o);
        const float w = exp2f(ml.x - m);
        l += w * ml.y;
#pragma unroll
        for (int e = 0; e < E; ++e) acc[e] += w * o[e];
    }
    if (mask != nullptr) {
        for (int cp = 0; cp < n_cand; ++cp) {
            if ((bits >> cp) & 1u) {
                const float w = exp2f(cs[cp] - m);
                float vr[E];
                load_run<E, BF16>(cvv, (((int64_t)i * n_cand + cp) * n_kv + hq / group) * D + c16 * E, vr);
                l += w;
#pragma unroll
                for (int e = 0; e < E; ++e) acc[e] += w * vr[e];
            }
        }
    }
    if (!ok) return;
    const float inv = 1.0f / l;
    const int64_t obase = (((int64_t)i * n_cand + c) * n_q + hq) * D + c16 * E;
    if constexpr (BF16) {
        uint32_t w[E / 2];
#pragma unroll
        for (int e = 0; e < E / 2; ++e)
            w[e] = (uint32_t)f32_to_bf16_rne(acc[2 * e] * inv) | ((uint32_t)f32_to_bf16_rne(acc[2 * e + 1] * inv) << 16);
        *reinterpret_cast<uint4*>(reinterpret_cast<uint16_t*>(outv) + obase) = uint4{w[0], w[1], w[2], w[3]};
    } else {
#pragma unroll
        for (int e = 0; e < E; e += 4)
            *reinterpret_cast<float4*>(reinterpret_cast<float*>(outv) + obase + e) =
                float4{acc[e] * inv, acc[e + 1] * inv, acc[e + 2] * inv, acc[e + 3] * inv};
    }
}

}  // namespace

// ---------------------------------------------------------------------------
// Fixed workspace of apar_decode_attention_fixed: the plan tables and the partial results of one call live
// in this array instead of in memory the library allocates.  Every GPU the library runs on holds its own
// copy of the array, at its own address, until the process ends.  In host code the array's name is only a
// handle of the symbol, not a device address: the address comes from hipGetSymbolAddress, once per device
// with that device current, and that pointer is what kernels and copies are given.
// ---------------------------------------------------------------------------
static __device__ __align__(256) unsigned char scratch[(size_t)APAR_FIXED_PLAN_BYTES + (size_t)APAR_FIXED_PARTIAL_BYTES];

namespace {
constexpr int kMaxDevices = 64;
char* g_scratch_ptr[kMaxDevices] = {};  // per device: where its copy of `scratch` lives (null: not asked yet)
}  // namespace

hipError_t fixed_workspace_of_device(int device, char** out) {
    if (device < 0 || device >= kMaxDevices || !out) return hipErrorInvalidValue;
    if (!g_scratch_ptr[device]) {
        void* ptr = nullptr;
        const hipError_t e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        if (!ptr || ((uintptr_t)ptr & 255)) return hipErrorInvalidSymbol;
        g_scratch_ptr[device] = (char*)ptr;
    }
    *out = g_scratch_ptr[device];
    return hipSuccess;
}

hipError_t launch_append_blocks(const Shape& s, void* pool, const void* k, const void* v, const int32_t* words, bool on_host,
                                int n_blocks, int n_open, int n_src, hipStream_t st) {
    if (n_blocks <= 0) return hipSuccess;
    if (s.dtype == APAR_F32 && n_open != n_blocks) return hipErrorInvalidValue;  // (fp32 blocks are never sealed)
    const int pairs = s.dtype == APAR_F32 && s.d == 128 ? 4 : 8;
    const int64_t grid = ((int64_t)n_open * s.n_kv + pairs - 1) / pairs + ((int64_t)(n_blocks - n_open) * s.n_kv + 3) / 4;
    if (grid > 0x7fffffff || (int64_t)n_blocks * s.n_kv > 0x7fffffff) return hipErrorInvalidValue;
    AppendTables<kAppendDevice> ptr{words};
    AppendTables<kAppendArguments> args;
    if (on_host && (size_t)4 * n_blocks + n_src > sizeof(args.words) / sizeof(int32_t)) {
        const AppendBlock* b = (const AppendBlock*)words;
        const int before = n_src == 0 ? append_run(b, n_blocks) : -1;
        if (before < 0 || s.dtype == APAR_F32) return hipErrorInvalidValue;
        AppendTables<kAppendRun> run;
        run.words[0] = before;
        run.words[1] = b[before].first;
        run.words[2] = run.words[3] = 0;
        memcpy(run.words + 4, b, before * sizeof(AppendBlock));
        for (int i = before; i < n_blocks; ++i) run.words[4 + 3 * before + i] = b[i].dst;
        if (s.fp8_sealed)
            hipLaunchKernelGGL((append_blocks<256, 2, kAppendRun>), dim3((unsigned)grid), dim3(256), 0, st, run, (char*)pool,
                               (const char*)k, (const char*)v, n_blocks, n_open, 0, s.n_kv);
        else
            hipLaunchKernelGGL((append_blocks<256, 1, kAppendRun>), dim3((unsigned)grid), dim3(256), 0, st, run, (char*)pool,
                               (const char*)k, (const char*)v, n_blocks, n_open, 0, s.n_kv);
        return hipGetLastError();
    }
    if (on_host) {
        for (int i = 0; i < 4 * n_blocks + n_src; ++i) args.words[i] = words[i];
    }
#define APAR_APPEND(ROWV, SEALV)                                                                                           \
    do {                                                                                                                   \
        if (on_host)                                                                                                       \
            hipLaunchKernelGGL((append_blocks<ROWV, SEALV, kAppendArguments>), dim3((unsigned)grid), dim3(256), 0, st, args,           \
                               (char*)pool, (const char*)k, (const char*)v, n_blocks, n_open, n_src, s.n_kv);                      \
        else                                                                                                               \
            hipLaunchKernelGGL((append_blocks<ROWV, SEALV, kAppendDevice>), dim3((unsigned)grid), dim3(256), 0, st, ptr,           \
                               (char*)pool, (const char*)k, (const char*)v, n_blocks, n_open, n_src, s.n_kv);                      \
    } while (0)
    if (s.dtype == APAR_F32) {
        if (s.d == 64) APAR_APPEND(256, 0);
        else APAR_APPEND(512, 0);
    } else if (s.fp8_sealed) {
        APAR_APPEND(256, 2);
    } else {
        APAR_APPEND(256, 1);
    }
#undef APAR_APPEND
    return hipGetLastError();
}

hipError_t launch_block_copies(const Shape& s, void* pool, const int32_t* pairs, int n_pairs, hipStream_t st) {
    if (n_pairs <= 0) return hipSuccess;
    int slices = (int)((s.block_bytes / 16 + 255) / 256);
    if (slices > 64) slices = 64;
    if (slices < 1) slices = 1;
    hipLaunchKernelGGL(copy_blocks, dim3(n_pairs, slices), dim3(256), 0, st, (char*)pool, pairs, s.block_bytes);
    return hipGetLastError();
}

// Bound by the host's memory over PCIe, and below some 100 KB by the launch.  A copy by the runtime goes to a DMA engine from
// 16 KiB on, which the kernels behind it wait some 20 us for (kernel to kernel beside a kernel of 70 us, copy by the runtime /
// this kernel: 4 and 16 KiB 4.9 / 5.1 us, 64 KiB 20.1 / 5.9, 200 KB 22.6 / 8.7, 1 MB 36.9 / 27.8).
__global__ __launch_bounds__(256) void copy_words(uint4* __restrict__ to, const uint4* __restrict__ from, int n) {
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i < n) to[i] = from[i];
}

hipError_t copy_staged(void* dev, const void* host, size_t bytes, hipStream_t st) {
    if (bytes == 0) return hipSuccess;
    const size_t n = (bytes + 15) / 16;
    if (n > 0x7fffffff - 255 || ((uintptr_t)dev | (uintptr_t)host) % 16 != 0) return hipErrorInvalidValue;
    hipLaunchKernelGGL(copy_words, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, (uint4*)dev, (const uint4*)host, (int)n);
    return hipGetLastError();
}

// words[pairs[2 i]] = pairs[2 i + 1]: brings staged plan tables up to date word by word, out of pinned host memory (a
// copy of its own first would be one more launch).  Pairs that name the same word carry the same value.
__global__ __launch_bounds__(256) void scatter_words(int32_t* __restrict__ words, const int32_t* __restrict__ pairs, int n) {
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i >= n) return;
    const int2 p = reinterpret_cast<const int2*>(pairs)[i];
    words[p.x] = p.y;
}

hipError_t launch_scatter_words(int32_t* words, const int32_t* pairs, int n_pairs, hipStream_t st) {
    if (n_pairs <= 0) return hipSuccess;
    hipLaunchKernelGGL(scatter_words, dim3((n_pairs + 255) / 256), dim3(256), 0, st, words, pairs, n_pairs);
    return hipGetLastError();
}

__global__ __launch_bounds__(256) void clear_words(int32_t* __restrict__ words, int n) {
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i < n) words[i] = 0;
}

hipError_t launch_clear_words(int32_t* words, int n, hipStream_t st) {
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(clear_words, dim3((n + 255) / 256), dim3(256), 0, st, words, n);
    return hipGetLastError();
}

hipError_t launch_read_rows(const Shape& s, const void* pool, const int32_t* src_codes, int n_rows, void* k_out,
                            void* v_out, hipStream_t st) {
    if (n_rows <= 0) return hipSuccess;
    dim3 grid(n_rows, s.n_kv);
    if (s.dtype == APAR_BF16)
        hipLaunchKernelGGL(read_rows_bf16, grid, dim3(64), 0, st, (const char*)pool, (uint16_t*)k_out,
                           (uint16_t*)v_out, src_codes, s.n_kv, s.tile_bytes, s.fp8_sealed);
    else
        hipLaunchKernelGGL(read_rows_f32, grid, dim3(64), 0, st, (const char*)pool, (float*)k_out, (float*)v_out,
                           src_codes, s.n_kv, s.d, s.tile_bytes);
    return hipGetLastError();
}

hipError_t launch_attention_partial(const Shape& s, const void* pool, const void* q, const PlanDev& plan, int n_cand,
                                    PartialBuf part, const void* cand_k, const void* cand_v, const uint8_t* mask,
                                    void* out, hipStream_t st) {
    if (plan.n_wg <= 0) return hipSuccess;
    if (s.dtype == APAR_BF16)
        return launch_attention_bf16(s, pool, q, plan, n_cand, part, cand_k, cand_v, mask, out, st);
    return launch_attention_f32(s, pool, q, plan, n_cand, part, cand_k, cand_v, mask, out, st);
}

hipError_t launch_merge(const Shape& s, const PlanDev& plan, PartialBuf part, const void* q, const void* cand_k,
                        const void* cand_v, const uint8_t* mask, int n_cand, void* out, hipStream_t st) {
    if (plan.n_threads <= 0) return hipSuccess;
    // grid.z carries the listed threads (limit 65535): go through them in slices
    const int kSlice = 32768;
    for (int i0 = 0; i0 < plan.n_threads; i0 += kSlice) {
        const int ni = plan.n_threads - i0 < kSlice ? plan.n_threads - i0 : kSlice;
        PlanDev pl = plan;
        pl.path_ofs = plan.path_ofs + i0;
        const int64_t e = s.dtype == APAR_F32 ? 4 : 2;
        const int64_t qofs = (int64_t)i0 * n_cand * s.n_q * s.d * e;
        const int64_t kofs = (int64_t)i0 * n_cand * s.n_kv * s.d * e;
        const void* q2 = (const char*)q + qofs;
        const void* ck2 = cand_k ? (const char*)cand_k + kofs : nullptr;
        const void* cv2 = cand_v ? (const char*)cand_v + kofs : nullptr;
        const uint8_t* mk2 = mask ? mask + (int64_t)i0 * n_cand : nullptr;
        void* out2 = (char*)out + qofs;
        dim3 grid((s.n_q + 15) / 16, n_cand, ni);
#define APAR_MERGE(DD, BF)                                                                                        \
    hipLaunchKernelGGL((merge_rows<DD, BF>), grid, dim3(256), 0, st, pl, part, q2, ck2, cv2, mk2, n_cand, s.n_q, \
                       s.n_kv, s.group, s.scale_log2e, out2)
        if (s.dtype == APAR_BF16) APAR_MERGE(128, true);
        else if (s.d == 64) APAR_MERGE(64, false);
        else APAR_MERGE(128, false);
#undef APAR_MERGE
    }
    return hipGetLastError();
}

}  // namespace apar
