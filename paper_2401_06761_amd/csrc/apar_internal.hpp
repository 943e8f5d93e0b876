// Internal declarations shared by the host side and the kernels of libapar.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "apar.h"

namespace apar {

constexpr int kBlockTokens = 16;
constexpr int32_t kCodeSealed = 1 << 30;  // flag on a (block * 16 + slot) code: the block is sealed
constexpr int64_t kMaxPoolBlocks = (int64_t)1 << 26;  // block * 16 + slot must stay below the flag bit
static_assert(kMaxPoolBlocks * kBlockTokens <= kCodeSealed, "a slot code must not reach the sealed flag");

// ---------------------------------------------------------------------------
// Pool layout in HBM.
//
// The pool is [block][kv_head] tiles; a tile holds the K rows and then the V
// rows of the block's 16 token slots for that head.
//
// f32 pools: both halves are row-major [16][d].
//
// bf16 pools (d = 128; tile = 4 KiB of K + 4 KiB of V).  A block that is still
// filling (fewer than 16 slots written) is row-major too, so that appending a row
// is a few full-line writes.  When its sixteenth slot is written the block is
// SEALED: both halves are rewritten in the order the 16x16 matrix-core
// instructions consume them, so that a wavefront fills its operand registers with
// four fully coalesced 1 KiB loads per half and no shuffle or LDS pass.  Full
// blocks are never written again, and every thread that holds a block agrees on
// its fill count, so "filled slots < 16" is all a reader needs to know the format.
// Sealed layout, with lane = 16*g + c (g = 0..3, c = 0..15) and load index
// r = 0..3: the 16 bytes at  r*1024 + lane*16  hold
//   K half: K[token c][dims 32*g + 8*r .. +8]               (A operand of K.Q^T)
//   V half: V[tokens 4*g .. 4*g+3][dim 32*r + c] followed by
//           V[tokens 4*g .. 4*g+3][dim 32*r + 16 + c]       (A operand of V^T.P^T)
//
// fp8 pools (APAR_BF16_FP8KV) seal a block into fp8 codes (OCP e4m3) in the same element order, one
// byte per element: the K half is bytes [0, 2048) of the tile, the V half [2048, 4096), and piece r
// of a lane is the 8 bytes at  half + (r/2)*1024 + lane*16 + (r%2)*8  (a 16-byte load brings two
// pieces).  Bytes [4096, 4104) hold two floats, the scale of the K half and of the V half: powers
// of two, value = code * scale.  The rest of the 8 KiB tile is unused while the block is sealed.
// ---------------------------------------------------------------------------
constexpr int kFp8HalfBytes = 2048;   // one half (K or V) of a sealed fp8 tile
constexpr int kFp8ScaleOfs = 4096;    // float K scale, float V scale
__host__ __device__ inline int fp8_k_offset(int token, int dim) {  // byte offset of an element inside the K half
    const int r = (dim & 31) >> 3, lane = (dim >> 5) * 16 + token;
    return (r >> 1) * 1024 + lane * 16 + (r & 1) * 8 + (dim & 7);
}
__host__ __device__ inline int fp8_v_offset(int token, int dim) {  // byte offset of an element inside the V half
    const int r = dim >> 5, lane = (token >> 2) * 16 + (dim & 15);
    return (r >> 1) * 1024 + lane * 16 + (r & 1) * 8 + ((dim >> 4) & 1) * 4 + (token & 3);
}
__host__ __device__ inline int bf16_k_offset(int token, int dim) {  // byte offset inside the K half
    return ((dim & 31) >> 3) * 1024 + (((dim >> 5) * 16 + token) * 16) + (dim & 7) * 2;
}
__host__ __device__ inline int bf16_v_offset(int token, int dim) {  // byte offset inside the V half
    return (dim >> 5) * 1024 + (((token >> 2) * 16 + (dim & 15)) * 16) + ((dim >> 4) & 1) * 8 + (token & 3) * 2;
}

// ---------------------------------------------------------------------------
// Plan tables (built on the host, read by the attention and merge kernels).
//
// The listed threads are numbered in depth-first order of their sharing tree, so
// the threads that hold any given block are a contiguous range of ranks.  A
// thread's query rows (candidates x q heads of one kv group) are cut into
// `n_slices` slices of at most 16 rows; (thread, slice) is a "row group" with
// index rank * n_slices + slice.  A wavefront holds up to row_tiles * (16 / rows_per_slice)
// consecutive row groups as the columns of its row_tiles 16x16 tiles (a row group
// never straddles two tiles: group j of the wavefront sits in tile j / (16 / rows_per_slice)).
// ---------------------------------------------------------------------------
struct TileRef {     // one block to read, and the row groups it applies to
    int32_t blk;
    int32_t meta;    // lo | hi << 10 | valid << 20: row groups [lo, hi) relative to the list owner's first
                     // row group (the workgroup's for shared lists, the wavefront's for its own list);
                     // valid = filled token slots (1..16).  Bit 30 marks a causal tile (prefill): row
                     // group lo sees only the first `first` slots (bits 25-29, 1..16), group lo + 1 one
                     // more, and so on up to valid.
};

// Most 16-row tiles one wavefront is given.  The kernels take 4 as well, but with 64 rows of state a
// wavefront runs out of the 256 architectural registers and the compiler shuttles accumulators to and
// from the accumulation registers around every use: measured slower than two tiles plus partial results
// (decode) or more workgroups (prefill), so the plans stop at 2.
constexpr int kMaxRowTiles = 2;
// Value of a workgroup descriptor's row-tile byte that marks a matrix unit (bf16 pools): a stand-alone
// chunk of a shared segment for up to 128 query rows, run by the 32x32 kernel.  Its shared tile list is
// the chunk; wavefront entry 0 names the threads (row groups of whole threads, rows laid flat over the
// workgroup) and the first thread's partial-result row; entries 1..3 are empty.
constexpr int kMatrixUnitRows = 32;
constexpr int kMatrixUnitMaxRows = 128;

struct WaveItem {    // what one wavefront computes
    int32_t tile_ofs, n_tiles;  // its own tile list
    int32_t grp_lo, n_grp;      // its row groups [grp_lo, grp_lo + n_grp); n_grp == 0: nothing to compute
    int32_t part_base;          // partial-result row of the thread that owns row group grp_lo
    int32_t flags;              // kWaveDirect: normalise and write the output rows instead of partial results
};
constexpr int32_t kWaveDirect = 1;
constexpr int32_t kWaveSplit = 2;  // the group's four wavefronts hold the SAME rows and a quarter of the tiles each;
                                   // their results are combined in LDS and wavefront 0 writes them
constexpr int kSplitMinTiles = 16; // shorter private units are packed four to a workgroup instead

// Every tile list holds its full tiles (16 filled slots) first and its open ones last, so that
// the kernels can run the bulk of a list through a loop that knows nothing of open tiles.
struct WgDesc {      // one 256-thread workgroup: a shared tile list, then one private list per wavefront
    int32_t coop_ofs, n_coop;   // tiles every wavefront of the group sees (staged once through LDS)
    int32_t grp_base;           // row group that the shared list's ranges are relative to
    int32_t row_tiles;          // bits 0-7: 16-row tiles per wavefront (1 or 2);
                                // bits 8-31: full shared tiles
    WaveItem w[4];
    int32_t n_full[4];          // full tiles at the head of each wavefront's own list
};
static_assert(sizeof(WgDesc) == 128, "WgDesc is read with aligned scalar loads");

// One workgroup (per kv head) of a launch some of whose units are cut into slices (attn_split.hpp).
struct SplitBlock {
    int32_t wg;               // the unit: index of its workgroup descriptor
    int32_t slice;            // slice | slices of the unit << 16
    int32_t state;            // where the unit's row states start, in 16-row tiles per kv head ...
    int32_t cut;              // ... and the unit's number among those that are cut
};
struct SplitPlan {
    const SplitBlock* blocks; // in launch order; null: no unit is cut and workgroups are units
    int32_t n_blocks_class[3];
    float* state;             // per cut unit: [kv head][slice][wavefront][row tile] states
    int32_t* arrived;         // per cut unit: [kv head][wavefront], zero between launches
};

struct PlanDev {              // device pointers of one staged plan
    const WgDesc* wgs;
    const TileRef* tiles;
    const int32_t* dfs_threads;  // rank -> index into the listed threads (null: the identity)
    const int32_t* path_ofs;     // [n_threads + 1], by listed index
    const int32_t* path_ids;     // partial-result rows to merge for each listed thread (none: written directly)
    int32_t n_wg;
    int32_t n_wg_class[3];       // matrix units, workgroups with 2 and with 1 row tiles per wavefront, stored in that order
    int32_t n_threads;
    int32_t rows_per_thread, rows_per_slice, n_slices;
    int32_t few;                 // 16-bit pools: the units go to the kernel for few workgroups; 2: its launcher packs inline_words
    SplitPlan split;
    const int32_t* inline_words; // small plans: the tables on the host, to go along with the kernel's arguments; every table
    int32_t n_inline_words;      // pointer above (split.blocks, always there then, included) is its offset in bytes
};

// Units of calls of few units, packed to go along with the kernel's arguments: two words per wavefront instead of a descriptor of 32, a word per
// tile.  Such units list shared blocks once each, and where their tables did not fit any more but the general plan's did, every step of a loop
// had a launch more than under that: of 70 drawn loops of that kind (a row per thread and step, 7 to 24 steps) 52 were slower than under the
// general plan, in the mean 1.10 times its time and five requests of six threads, group 8, 1.28 times; packed 3, 0.85 and 1.02.
// Blocks have 18 bits; larger pools send the tables as they are.  The other fields hold whatever fits kPlanInlineWords: less than 1024 tiles, at
// most 832 threads of up to four slices, 32 row groups per unit.
constexpr int64_t kFewPackedBlocks = 1 << 18;
constexpr int kFewWaveWords = 2;
inline size_t few_packed_words(size_t n_wg, size_t n_blocks, size_t n_tiles, size_t n_threads) {
    return n_wg * 4 * kFewWaveWords + n_blocks * (sizeof(SplitBlock) / 4) + n_tiles + n_threads;
}
__host__ __device__ inline uint32_t pack_few_tile(const TileRef& t) {
    return (uint32_t)t.blk << 14 | (t.meta & 31) << 9 | (((t.meta >> 10) - 1) & 31) << 4 | (((t.meta >> 20) - 1) & 15);
}
__host__ __device__ inline TileRef unpack_few_tile(uint32_t w) {
    return TileRef{(int32_t)(w >> 14), (int32_t)((w >> 9 & 31) | ((w >> 4 & 31) + 1) << 10 | ((w & 15) + 1) << 20)};
}
__host__ __device__ inline void pack_few_wave(const WaveItem& wi, int n_full, uint32_t (&w)[kFewWaveWords]) {
    w[0] = (uint32_t)((wi.tile_ofs & 1023) | wi.n_tiles << 10 | (n_full < wi.n_tiles ? n_full : wi.n_tiles) << 20);
    w[1] = (uint32_t)((wi.grp_lo & 4095) | wi.n_grp << 12 | wi.flags << 18);
}
__host__ __device__ inline WaveItem unpack_few_wave(uint32_t w0, uint32_t w1, int& n_full) {
    n_full = (int)(w0 >> 20);
    return WaveItem{(int32_t)(w0 & 1023), (int32_t)(w0 >> 10 & 1023), (int32_t)(w1 & 4095), (int32_t)(w1 >> 12 & 63), 0, (int32_t)(w1 >> 18)};
}

// The first argument of the attention kernels; they take it from the head of the argument segment.
constexpr int kPlanInlineWords = 832;
template <bool INLINE>
struct PlanWords {
    const int32_t* unused;
};
template <>
struct PlanWords<true> {
    int32_t words[kPlanInlineWords];
};
#if defined(__HIP_DEVICE_COMPILE__)
// A plan whose tables are the kernel's first argument.
__device__ __forceinline__ void plan_from_arguments(PlanDev& plan) {
    const char* base = (const char*)(const char __attribute__((address_space(4)))*)__builtin_amdgcn_kernarg_segment_ptr();
    plan.wgs = (const WgDesc*)(base + (size_t)plan.wgs);
    plan.tiles = (const TileRef*)(base + (size_t)plan.tiles);
    plan.dfs_threads = (const int32_t*)(base + (size_t)plan.dfs_threads);
    plan.split.blocks = (const SplitBlock*)(base + (size_t)plan.split.blocks);
}
// A table that no kernel writes.  A kernel that runs either of two bodies tells the compiler so: control flow is put in order
// before loads are chosen, the second body then lies behind the first one's stores, and the words of its lists would be
// fetched by vector loads, each of which waits for all tiles in flight (multi-candidate call of 20.7 k threads, 32 heads: 14.0 ms
// instead of 11.7).
template <class T>
__device__ __forceinline__ const T* unwritten(const T* p) {
    auto c = (const T __attribute__((address_space(4)))*)p;
    asm("" : "+s"(c));
    return (const T*)c;
}
__device__ __forceinline__ void tables_unwritten(PlanDev& plan) {
    plan.wgs = unwritten(plan.wgs);
    plan.tiles = unwritten(plan.tiles);
    plan.dfs_threads = unwritten(plan.dfs_threads);
}
#elif defined(__HIP__)
__device__ inline void plan_from_arguments(PlanDev&) {}
__device__ inline void tables_unwritten(PlanDev&) {}
template <class T>
__device__ inline const T* unwritten(const T* p) { return p; }
#endif

struct PrefillWg {            // one workgroup of the bf16 prefill kernel: consecutive query tokens of one thread
    int32_t table_ofs;        // the thread's block table inside the staged tables
    int32_t q_row0;           // index of its first query token among the call's query tokens
    int32_t p0;               // position of that token in the thread
    int32_t n_tok;            // query tokens it holds (n_tok * group <= 128 rows)
    int32_t len;              // the thread's length
    int32_t pad[3];
};
static_assert(sizeof(PrefillWg) == 32, "PrefillWg is read with one aligned scalar load");

struct Shape {
    int32_t n_q, n_kv, d, group;  // group = n_q / n_kv
    int32_t dtype;                // element type of rows at the interface and in blocks that are still filling: APAR_F32 or APAR_BF16
    int32_t fp8_sealed;           // 1: full blocks are kept in fp8 with a power-of-two scale per (block, kv head) and half
    float scale_log2e;            // softmax scale * log2(e): logits are kept in base 2
    int64_t tile_bytes;           // one (block, kv head): 2 * 16 * d * e
    int64_t block_bytes;          // n_kv tiles
};

// One block an append call writes to.
struct AppendBlock {
    int32_t dst;
    int32_t copy_of;          // the shared block whose rows before the first new one it takes over (copy on write), or -1
    int32_t first;            // source row of the first new row, or, with a list of source rows, its place in the list
    int32_t slots;            // new rows: slots [slots & 255, slots >> 8)
};
static_assert(sizeof(AppendBlock) == 16, "four words of the staged tables");
constexpr int kAppendInlineWords = 480;
// Most blocks of a long append are a run: whole, in the order of the source rows.  Of those only the block goes along: words 0 and 1
// are the number of the blocks before the run and the run's first source row, then come the former (from word 4) and the run.
constexpr int kAppendRunWords = 960, kAppendRunMaxBefore = 8;
// Where the run starts that ends a call's blocks, or -1 if they do not fit that way.
inline int append_run(const AppendBlock* b, int n) {
    int at = n;
    while (at > 0 && b[at - 1].slots == 16 << 8 && b[at - 1].copy_of < 0 && (at == n || b[at - 1].first + 16 == b[at].first)) --at;
    return at < n && at <= kAppendRunMaxBefore && 4 + 4 * at + (n - at) <= kAppendRunWords ? at : -1;
}
// Where an append's descriptors and source rows are: on the device, or the kernel's first argument, all of them or as a run.
enum AppendFrom { kAppendDevice, kAppendArguments, kAppendRun };
template <int FROM>
struct AppendTables {
    int32_t words[FROM == kAppendRun ? kAppendRunWords : kAppendInlineWords];
};
template <>
struct AppendTables<kAppendDevice> {
    const int32_t* words;
};

// Partial results: for partial row p, candidate c, q head h the slot is
// (p * n_cand + c) * n_q + h; part_o holds d floats per slot, part_ml two (max, sum).
struct PartialBuf {
    float* o;
    float* ml;
    int32_t stream;  // this call's are more than the memory-side cache holds: written with non-temporal stores
};
// Measured (bf16; attention + merge, us, plain / non-temporal stores; partial rows x 32 heads of 520 bytes each):
// 20 rows (32 k tokens, 4 threads) 33.6 + 8.0 / 33.6 + 9.4, 1547 rows (26 MB) 247 + 10 / 249 + 12, 13 k rows (218 MB)
// 1827 + 41 / 1813 + 49, 50 k rows (831 MB) 3758 + 179 / 3675 + 173; 1600 rows of matrix units 186 + 10 / 188 + 11.
constexpr size_t kStreamPartialBytes = (size_t)256 << 20;

// The most room for the row states of a launch some of whose units are cut into slices (attn_split.hpp), a pool has an eighth of its own size up
// to this: 256 shares of a 16-bit call's work are fewer than 512 slices x kv heads, of at most 8 row tiles of 8.5 KiB.  fp32 calls may want
// more (512 shares, or up to 64 slices a unit by an estimate): cut_into_slices makes slices longer until they fit.
// kSplitMaxCut: the most cut units x kv heads, which it keeps to in the same way.
constexpr size_t kSplitStateBytes = (size_t)32 << 20;
constexpr int kSplitMaxCut = 512;
constexpr size_t kSplitCounterBytes = (size_t)kSplitMaxCut * 4 * sizeof(int32_t);

// Where `device`'s copy of the library's static workspace (APAR_FIXED_PLAN_BYTES of plan tables followed by
// APAR_FIXED_PARTIAL_BYTES of partial results) lives.  `device` must be the current device.  The address is
// asked for once per device and kept.
hipError_t fixed_workspace_of_device(int device, char** out);

// ---- launchers (defined next to their kernels) ------------------------------
// words: n_blocks AppendBlocks, the n_open that stay open first, then n_src source rows; on the host (at most kAppendInlineWords words, or,
// without source rows on 16-bit pools, blocks that append_run takes, which go along with the kernel's arguments) or on the device.
hipError_t launch_append_blocks(const Shape& s, void* pool, const void* k, const void* v, const int32_t* words, bool on_host,
                                int n_blocks, int n_open, int n_src, hipStream_t st);
hipError_t launch_block_copies(const Shape& s, void* pool, const int32_t* src_dst_pairs, int n_pairs,
                               hipStream_t st);
// Staged tables, from pinned host memory to the device (both 16-byte aligned, and padded to 16 bytes), by a kernel.
#if defined(__HIP__)
hipError_t copy_staged(void* dev, const void* host, size_t bytes, hipStream_t st);
#else  // a build of the host side alone has no kernels
inline hipError_t copy_staged(void* dev, const void* host, size_t bytes, hipStream_t st) {
    return hipMemcpyAsync(dev, host, bytes, hipMemcpyHostToDevice, st);
}
#endif
// words[pairs[2 i]] = pairs[2 i + 1] for i < n_pairs (words on the device, pairs in pinned host memory, 8-byte aligned)
hipError_t launch_scatter_words(int32_t* words, const int32_t* pairs, int n_pairs, hipStream_t st);
// words[i] = 0 for i < n
hipError_t launch_clear_words(int32_t* words, int n, hipStream_t st);
hipError_t launch_read_rows(const Shape& s, const void* pool, const int32_t* src_codes, int n_rows, void* k_out,
                            void* v_out, hipStream_t st);
hipError_t launch_attention_partial(const Shape& s, const void* pool, const void* q, const PlanDev& plan, int n_cand,
                                    PartialBuf part, const void* cand_k, const void* cand_v, const uint8_t* mask,
                                    void* out, hipStream_t st);
hipError_t launch_attention_bf16(const Shape& s, const void* pool, const void* q, const PlanDev& plan, int n_cand,
                                 PartialBuf part, const void* cand_k, const void* cand_v, const uint8_t* mask,
                                 void* out, hipStream_t st);
hipError_t launch_attention_few_bf16(const Shape& s, const void* pool, const void* q, const PlanDev& plan, int n_cand, PartialBuf part,
                                     const void* cand_k, const void* cand_v, const uint8_t* mask, void* out, hipStream_t st);
hipError_t launch_attention_f32(const Shape& s, const void* pool, const void* q, const PlanDev& plan, int n_cand,
                                PartialBuf part, const void* cand_k, const void* cand_v, const uint8_t* mask, void* out,
                                hipStream_t st);
hipError_t launch_prefill_bf16(const Shape& s, const void* pool, const void* q, const PrefillWg* wgs,
                               const int32_t* tables, int n_wg, void* out, hipStream_t st);
// workgroups [wg_first, wg_first + n_wg) of the plan: matrix units (row_tiles byte = kMatrixUnitRows)
hipError_t launch_attention_units_bf16(const Shape& s, const void* pool, const void* q, const PlanDev& plan,
                                       int wg_first, int n_wg, int n_cand, PartialBuf part, hipStream_t st);
hipError_t launch_merge(const Shape& s, const PlanDev& plan, PartialBuf part, const void* q, const void* cand_k,
                        const void* cand_v, const uint8_t* mask, int n_cand, void* out, hipStream_t st);


}  // namespace apar
