// Host side of libapar: the C ABI, the block/refcount/fork bookkeeping, the
// plan builder that groups threads by the blocks they share, and the staging of
// small tables to the device.  Every device step runs in the HIP kernels; this
// file only decides which blocks they touch.
#include <algorithm>
#include <chrono>
#include <cmath>
#include <cstdio>
#include <cstring>
#include <new>
#include <string>
#include <unordered_map>
#include <vector>

#include "apar_internal.hpp"
#include "plan.hpp"

using namespace apar;

namespace {

thread_local std::string g_last_hip_error;

bool hip_ok(hipError_t e, const char* what) {
    if (e == hipSuccess) return true;
    g_last_hip_error = std::string(what) + ": " + hipGetErrorString(e);
    (void)hipGetLastError();  // (reported here: the next launch's check must not find it)
    return false;
}
#define HIP_TRY(expr)                                  \
    do {                                               \
        if (!hip_ok((expr), #expr)) return APAR_ERR_HIP; \
    } while (0)

struct Thread {
    bool live = false;
    int32_t forked_from = -1;  // the thread it was forked from (kept after either is released)
    int64_t len = 0;
    std::vector<int32_t> table;
};

// A pinned host buffer and its device twin, reused round-robin.  The event marks
// the last device work that read the pair, so a slot is only rewritten after it.
struct StageSlot {
    char* host = nullptr;
    char* dev = nullptr;
    size_t cap = 0;
    hipEvent_t ev = nullptr;   // recorded after the kernels that read the slot
    hipEvent_t up = nullptr;   // recorded after the slot's upload
    bool pending = false;
    bool own = false;          // the pair was allocated when the slot grew (else it is a part of the pool's workspace)
};
constexpr int kStageSlots = 4;
constexpr size_t kStageBytes = (size_t)1 << 20;  // what a slot holds to begin with
constexpr size_t kCopyStreamMinBytes = 256 << 10;  // uploads from this size on run on the pool's copy stream

struct EventPair {
    hipEvent_t a = nullptr, b = nullptr, c = nullptr;  // a..b first kernel(s), b..c second (c may be null)
};

inline size_t align_up(size_t x, size_t a) { return (x + a - 1) / a * a; }

constexpr size_t kFixedPlanBytes = (size_t)APAR_FIXED_PLAN_BYTES;
constexpr size_t kFixedPartBytes = (size_t)APAR_FIXED_PARTIAL_BYTES;

}  // namespace

struct apar_pool {
    apar_pool_config cfg{};
    Shape shape{};
    char* kv = nullptr;
    int device = 0;
    bool dry_run = false;  // bookkeeping and planning only: no device memory, nothing is launched

    std::vector<int32_t> ref;
    std::vector<int32_t> free_stack;
    std::vector<Thread> threads;  // index = thread id
    int64_t live_threads = 0;
    int64_t cow_copies = 0;

    // plan builder scratch (pool sized, kept clean between calls)
    std::vector<int32_t> seg_of;  // segment that starts at each block, -1 if none
    int max_unit_tiles = 512;  // longest tile list given to one wavefront
    int prefill_kernel = APAR_PREFILL_AUTO;
    // stand-alone segments with at least this many query rows and blocks run as matrix units (bf16 pools)
    int matrix_min_rows = 256, matrix_min_blocks = 128;
    bool inline_shared = true;  // subtrees with too many rows are cut by rank into direct units instead of leaving partial results
    bool has_matrix_units() const { return shape.dtype == APAR_BF16 && !shape.fp8_sealed; }  // (the 32x32 kernels read bf16 tiles only)
    bool check_writes = false;  // verify before every launch that no destination block is shared
    int last_prefill_kernel = 0;  // which kernel the most recent prefill call ran (APAR_PREFILL_ROW_TILES / _MATRIX)
    std::vector<PlanThreadView> views;
    std::vector<PrefillThreadView> prefill_views;
    std::vector<PrefillWg> prefill_wgs;
    std::vector<int32_t> prefill_tables;
    std::vector<int32_t> scratch_codes, scratch_copies, scratch_seals, scratch_commit_src;
    std::vector<apar_thread> scratch_commit_ids;
    std::vector<AppendBlock> append_blocks;
    std::vector<int32_t> append_of, append_src, append_words;
    apar_plan_info last_plan{};
    PlanHost plan;  // the last plan, kept for the next call to carry over, for reuse of its storage and for inspection
    // the call that plan was made or last carried over for: its listed threads, its parameters, and how many
    // threads the pool had ever created by then (a thread with an id from there on was forked since)
    std::vector<apar_thread> plan_ids;
    PlanParams plan_prm{};
    size_t plan_threads_then = 0;
    int64_t plan_copies_then = 0;  // copy-on-write copies the pool had made by then
    bool plan_reuse = true;
    int64_t n_plans_built = 0, n_plans_carried = 0;
    bool planning_set = false;         // one of the planner's knobs was set: plans are built as told, none for few units
    int32_t plan_geom[3] = {1, 1, 1};  // rows per thread, rows per slice, slices of the last plan

    StageSlot stage[kStageSlots];
    int next_slot = 0;
    size_t stage_want = 0;  // the largest staging request so far
    // The staging slot whose device half holds the tables of `plan`, as long as that is so: a call that carries
    // the plan over rewrites the changed words there instead of staging every table again.  Kept out of the
    // rotation meanwhile.  resident_behind: the host tables have moved on and the slot has not caught up yet
    // (set while a call is between the two; a call that fails there leaves it set and the slot is dropped).
    StageSlot* resident = nullptr;
    size_t resident_bytes = 0;
    bool resident_behind = false;
    PartialBuf part{};
    size_t part_slots_cap = 0;
    hipStream_t copy_stream = nullptr;  // uploads of plans and row codes run here, beside the caller's stream

    // Obtained at pool creation, an allocation each: pinned host memory (the buffer apar_decode_attention_fixed stages its
    // plan in, then the host halves of the staging slots), and device memory (counters and row states of launches whose
    // units are cut into slices, then the device halves of the staging slots).
    char* work_host = nullptr;
    char* work_dev = nullptr;

    // apar_decode_attention_fixed: this device's copy of the static workspace, the pinned host buffer the plan
    // is staged in, and the event after its upload
    char* fixed_dev = nullptr;
    char* fixed_host = nullptr;
    hipEvent_t fixed_up = nullptr;
    bool fixed_pending = false;

    // row states of launches whose units are cut into slices, behind the counters of slices that have arrived (zero
    // between launches once split_clear: a clear has run or is enqueued before any launch to come)
    char* split_dev = nullptr;
    size_t split_bytes = 0;
    bool split_clear = false;
    std::vector<SplitBlock> split_blocks;  // of the plan as it was built
    int32_t n_split_class[3] = {0, 0, 0};
    std::vector<int32_t> inline_words;  // a small plan's tables, as they go along with the kernels' arguments
    size_t inline_ofs[4] = {0, 0, 0, 0};

    bool profiling = false;
    std::vector<EventPair> decode_events, append_events;
    std::vector<hipEvent_t> spare_events;
    std::vector<float> last_attention_ms;  // per call, from the last profile read
    double plan_host_ms = 0.0, host_wait_ms = 0.0, wait_in_call_ms = 0.0;
    int64_t n_decode_calls = 0, n_append_calls = 0;
};

namespace {

struct DeviceGuard {
    int prev = 0;
    bool switched = false;
    explicit DeviceGuard(int dev) {
        if (hipGetDevice(&prev) == hipSuccess && prev != dev) switched = (hipSetDevice(dev) == hipSuccess);
    }
    ~DeviceGuard() {
        if (switched) (void)hipSetDevice(prev);
    }
};

Thread* live_thread(apar_pool* p, apar_thread t) {
    if (t < 0 || (size_t)t >= p->threads.size() || !p->threads[t].live) return nullptr;
    return &p->threads[t];
}

int32_t pop_block(apar_pool* p) {
    int32_t b = p->free_stack.back();
    p->free_stack.pop_back();
    p->ref[b] = 1;
    return b;
}

int grow_slot(StageSlot& s, size_t bytes) {
    if (s.own && s.host) HIP_TRY(hipHostFree(s.host));
    if (s.own && s.dev) HIP_TRY(hipFree(s.dev));
    s.host = s.dev = nullptr;
    s.cap = 0;
    s.own = true;
    const size_t cap = align_up(std::max(bytes + bytes / 2, kStageBytes), 4096);
    HIP_TRY(hipHostMalloc((void**)&s.host, cap, hipHostMallocDefault));
    HIP_TRY(hipMalloc((void**)&s.dev, cap));
    s.cap = cap;
    return APAR_OK;
}

// Everything a pool's calls work in besides the pool: all staging slots, so that no call of a loop stops to set one up
// (measured, one after the other: the third and fourth call of a new pool took 60 to 80 us on the host against 17), in one
// pinned and one device allocation.  Nothing is enqueued, so that creating a pool waits for nobody's work: the first launch
// with a cut unit clears the counters.
// A pool does without all of this but the buffer of apar_decode_attention_fixed, whose calls may not allocate: where memory
// is short, slots are set up by the calls that need them and no unit is cut.
int set_up_workspace(apar_pool* p, size_t pool_bytes) {
    if (!hip_ok(fixed_workspace_of_device(p->device, &p->fixed_dev), "hipGetSymbolAddress(scratch)")) return APAR_ERR_HIP;
    const size_t state_bytes = std::min(kSplitStateBytes, std::max((size_t)1 << 20, pool_bytes / 8));
    const size_t split = kSplitCounterBytes + state_bytes;
    if (hipMalloc((void**)&p->work_dev, split + kStageSlots * kStageBytes) == hipSuccess) {
        p->split_dev = p->work_dev;
        p->split_bytes = state_bytes;
    } else {
        (void)hipGetLastError();
        p->work_dev = nullptr;
    }
    if (hipHostMalloc((void**)&p->work_host, kFixedPlanBytes + kStageSlots * kStageBytes, hipHostMallocDefault) == hipSuccess) {
        for (int k = 0; p->work_dev && k < kStageSlots; ++k) {
            p->stage[k].host = p->work_host + kFixedPlanBytes + k * kStageBytes;
            p->stage[k].dev = p->work_dev + split + k * kStageBytes;
            p->stage[k].cap = kStageBytes;
        }
    } else {
        (void)hipGetLastError();
        HIP_TRY(hipHostMalloc((void**)&p->work_host, kFixedPlanBytes, hipHostMallocDefault));
    }
    p->fixed_host = p->work_host;
    HIP_TRY(hipEventCreateWithFlags(&p->fixed_up, hipEventDisableTiming));
    for (StageSlot& s : p->stage) HIP_TRY(hipEventCreateWithFlags(&s.ev, hipEventDisableTiming));
    return APAR_OK;
}

void release_workspace(apar_pool* p) {
    for (StageSlot& s : p->stage) {
        if (s.own && s.host) (void)hipHostFree(s.host);
        if (s.own && s.dev) (void)hipFree(s.dev);
        if (s.ev) (void)hipEventDestroy(s.ev);
        if (s.up) (void)hipEventDestroy(s.up);
    }
    if (p->work_host) (void)hipHostFree(p->work_host);
    if (p->work_dev) (void)hipFree(p->work_dev);
    if (p->fixed_up) (void)hipEventDestroy(p->fixed_up);
}

int acquire_stage(apar_pool* p, size_t bytes, StageSlot** out) {
    if (&p->stage[p->next_slot] == p->resident) p->next_slot = (p->next_slot + 1) % kStageSlots;
    StageSlot& s = p->stage[p->next_slot];
    p->next_slot = (p->next_slot + 1) % kStageSlots;
    if (s.pending) {
        const auto w0 = std::chrono::steady_clock::now();
        HIP_TRY(hipEventSynchronize(s.ev));
        s.pending = false;
        p->wait_in_call_ms = std::chrono::duration<double, std::milli>(std::chrono::steady_clock::now() - w0).count();
        if (p->profiling) p->host_wait_ms += p->wait_in_call_ms;
    }
    // Growing a slot frees device memory, which waits for the GPU to drain: a slot grows to what the largest
    // request so far would need, not just to this one, so that the slots of a loop whose calls alternate
    // between small and large tables (row codes, plan updates) stop growing after one round.
    p->stage_want = std::max(p->stage_want, bytes);
    if (s.cap < bytes) {
        const int rc = grow_slot(s, p->stage_want);
        if (rc != APAR_OK) return rc;
    }
    *out = &s;
    return APAR_OK;
}

// Uploads the first `bytes` of a staging slot on the pool's own copy stream and makes the caller's stream wait
// for it: the copy then runs beside whatever the caller's stream is still busy with (the previous step's
// attention, typically) instead of queueing behind it.  The slot is free by construction: acquire_stage waited
// for the kernels that last read it.
int upload(apar_pool* p, StageSlot* s, size_t bytes, hipStream_t st) {
    // Small tables go on the caller's stream, copied by a kernel: the hop to the copy stream and back costs more than it hides
    // when a step is a few launches long (a serving loop at a few hundred threads: 0.18 ms per step with the hop, 0.12
    // without), and a copy by the runtime keeps the kernels behind it waiting (a new plan every call: 64 requests, 32
    // heads 307 -> 295 us, one thread family of 32 k tokens 52 -> 41; figures per size beside copy_words).
    if (bytes < kCopyStreamMinBytes) {
        HIP_TRY(copy_staged(s->dev, s->host, bytes, st));
        return APAR_OK;
    }
    if (!p->copy_stream) HIP_TRY(hipStreamCreateWithFlags(&p->copy_stream, hipStreamNonBlocking));
    if (!s->up) HIP_TRY(hipEventCreateWithFlags(&s->up, hipEventDisableTiming));
    HIP_TRY(hipMemcpyAsync(s->dev, s->host, bytes, hipMemcpyHostToDevice, p->copy_stream));
    HIP_TRY(hipEventRecord(s->up, p->copy_stream));
    HIP_TRY(hipStreamWaitEvent(st, s->up, 0));
    return APAR_OK;
}

int new_event(apar_pool* p, hipEvent_t* ev) {
    if (!p->spare_events.empty()) {
        *ev = p->spare_events.back();
        p->spare_events.pop_back();
        return APAR_OK;
    }
    HIP_TRY(hipEventCreate(ev));
    return APAR_OK;
}

// Where token slot `pos` of a thread lives: block * 16 + slot.
inline int32_t slot_code(const Thread& t, int64_t pos) {
    return t.table[pos / kBlockTokens] * kBlockTokens + (int32_t)(pos % kBlockTokens);
}

// Advances one thread by one token following the allocator policy; the caller
// has already made sure enough free blocks exist.
inline int32_t append_one(apar_pool* p, Thread& t, std::vector<int32_t>& copies, std::vector<int32_t>& seals) {
    const int slot = (int)(t.len % kBlockTokens);
    if (slot == 0) {
        t.table.push_back(pop_block(p));
    } else {
        const int32_t tail = t.table.back();
        if (p->ref[tail] > 1) {  // shared, partly filled tail: copy on write
            const int32_t fresh = pop_block(p);
            copies.push_back(tail);
            copies.push_back(fresh);
            p->ref[tail] -= 1;
            t.table.back() = fresh;
            p->cow_copies += 1;
        }
    }
    const int32_t code = t.table.back() * kBlockTokens + slot;
    if (slot == kBlockTokens - 1) seals.push_back(t.table.back());  // the block is full after this row
    t.len += 1;
    return code;
}

// Write check (apar_set_write_checks): every block about to be written - appended rows, destinations of
// copy-on-write copies, blocks about to be re-laid-out - must be held by exactly one thread.
int writes_are_private(const apar_pool* p, const std::vector<int32_t>& codes, const std::vector<int32_t>& copies,
                       const std::vector<int32_t>& seals) {
    for (int32_t c : codes)
        if (p->ref[c / kBlockTokens] != 1) return APAR_ERR_INTERNAL;
    for (size_t i = 0; i + 1 < copies.size(); i += 2)
        if (p->ref[copies[i + 1]] != 1 || copies[i] == copies[i + 1]) return APAR_ERR_INTERNAL;
    for (int32_t b : seals)
        if (p->ref[b] != 1) return APAR_ERR_INTERNAL;
    return APAR_OK;
}

// Writes the call's rows: row i to codes[i], taken from row src_rows[i] of k, v (row i if src_rows is null), one
// AppendBlock per block written to.  A block is written by one thread only, whose rows fill its slots in order, but the
// thread may be listed in several places: the block's rows are contiguous in the call or get a list of source rows.
int run_append(apar_pool* p, const std::vector<int32_t>& codes, const std::vector<int32_t>& copies,
               const std::vector<int32_t>* src_rows, const void* k, const void* v, hipStream_t st) {
    std::vector<AppendBlock>& blocks = p->append_blocks;
    std::vector<int32_t>& at = p->append_of;  // per block of the pool: its place in `blocks` (-1 between calls)
    std::vector<int32_t>& src = p->append_src;
    blocks.clear();
    src.clear();
    bool contiguous = src_rows == nullptr;
    const int n = (int)codes.size();
    for (int i = 0; i < n; ++i) {
        const int32_t block = codes[i] / kBlockTokens, slot = codes[i] % kBlockTokens;
        int32_t& b = at[block];
        if (b < 0) {
            b = (int32_t)blocks.size();
            blocks.push_back(AppendBlock{block, -1, i, slot | (slot + 1) << 8});
        } else {
            AppendBlock& ab = blocks[b];
            contiguous = contiguous && i == ab.first + (ab.slots >> 8) - (ab.slots & 255);
            ab.slots += 1 << 8;
        }
    }
    if (!contiguous) {  // source rows, block by block
        int32_t ofs = 0;
        for (AppendBlock& b : blocks) {
            b.first = ofs;
            ofs += (b.slots >> 8) - (b.slots & 255);
        }
        src.resize(n);
        for (int i = 0; i < n; ++i) {
            const AppendBlock& b = blocks[at[codes[i] / kBlockTokens]];
            src[b.first + codes[i] % kBlockTokens - (b.slots & 255)] = src_rows ? (*src_rows)[i] : i;
        }
    }
    // Copy on write: the copy takes its first rows from the shared block as it is written.  A shared block that its last
    // holder fills and seals in this very call would change under its readers: then the copies are made first.
    bool copies_first = false;
    for (size_t i = 0; i + 1 < copies.size(); i += 2)
        copies_first = copies_first || (at[copies[i]] >= 0 && blocks[at[copies[i]]].slots >> 8 == kBlockTokens);
    if (!copies_first)
        for (size_t i = 0; i + 1 < copies.size(); i += 2) blocks[at[copies[i + 1]]].copy_of = copies[i];
    for (const AppendBlock& b : blocks) at[b.dst] = -1;
    int n_open = (int)blocks.size();  // the blocks that are not sealed come first
    const size_t words = blocks.size() * 4 + src.size();
    const size_t copy_words = copies_first ? copies.size() : 0;
    bool inlined = words <= (size_t)kAppendInlineWords && copy_words == 0;
    if (p->shape.dtype != APAR_F32) {
        auto stays_open = [](const AppendBlock& b) { return b.slots >> 8 < kBlockTokens; };
        const bool maybe_run = !inlined && copy_words == 0 && src.empty();
        n_open = (int)((maybe_run ? std::stable_partition(blocks.begin(), blocks.end(), stays_open)
                                  : std::partition(blocks.begin(), blocks.end(), stays_open)) -
                       blocks.begin());
        inlined = inlined || (maybe_run && append_run(blocks.data(), (int)blocks.size()) >= 0);
    }
    const int32_t* tables = (const int32_t*)blocks.data();
    StageSlot* s = nullptr;
    int rc = APAR_OK;
    if (inlined) {
        if (!src.empty()) {
            p->append_words.assign(tables, tables + blocks.size() * 4);
            p->append_words.insert(p->append_words.end(), src.begin(), src.end());
            tables = p->append_words.data();
        }
    } else {
        const size_t total = (words + copy_words) * sizeof(int32_t);
        if ((rc = acquire_stage(p, total, &s)) != APAR_OK) return rc;
        int32_t* host = (int32_t*)s->host;
        memcpy(host, blocks.data(), blocks.size() * sizeof(AppendBlock));
        if (!src.empty()) memcpy(host + blocks.size() * 4, src.data(), src.size() * sizeof(int32_t));
        if (copy_words) memcpy(host + words, copies.data(), copy_words * sizeof(int32_t));
        if ((rc = upload(p, s, total, st)) != APAR_OK) return rc;
        tables = (const int32_t*)s->dev;
    }
    EventPair ev;
    if (p->profiling) {
        if ((rc = new_event(p, &ev.a)) != APAR_OK || (rc = new_event(p, &ev.b)) != APAR_OK) return rc;
        HIP_TRY(hipEventRecord(ev.a, st));
    }
    if (copy_words) HIP_TRY(launch_block_copies(p->shape, p->kv, tables + words, (int)(copy_words / 2), st));
    HIP_TRY(launch_append_blocks(p->shape, p->kv, k, v, tables, inlined, (int)blocks.size(), n_open, (int)src.size(), st));
    if (p->profiling) {
        HIP_TRY(hipEventRecord(ev.b, st));
        p->append_events.push_back(ev);
        p->n_append_calls += 1;
    }
    if (s) {
        HIP_TRY(hipEventRecord(s->ev, st));
        s->pending = true;
    }
    return APAR_OK;
}

// Calls of few units: units of one row tile (or two) without shared lists, which the planner makes for them (PlanParams::few_units).  On 16-bit
// pools they go to a kernel of their own (attend_few): the shared lists of wider units cost a microsecond per tile where
// nobody else is there to fill the waits.  Measured, us per call (general plan and kernel / units of 16 rows and that kernel):
//   one request of 5 threads, group 1 11.7 / 8.4, group 4 14.4 / 8.2, two fork levels, group 4 17.4 / 9.4, of 9 threads of 24 rows each 49.5 / 14.6;
//   four requests, group 1 21.4 / 18.0, group 4 19.1 / 11.7, two fork levels 30.7 / 15.2; 16 requests, group 4 28.0 / 24.5, of 2 k tokens on
//   fp8 40.0 / 29.1; by units x kv heads: 292 40.5 / 25.5, 440 41.7 / 23.8, 472 47.0 / 43.2, 584 116.9 / 104.8, 720 32.4 / 26.8, 792 26.4 / 14.9, 824 44.6 / 37.0,
//   848 45.1 / 31.8; 2048 and more of whole trees 215.2 / 216.4.
// A tree of more rows than a unit holds is read by several units, from L2 at best, so that units have 32 rows where units of 16 would read
// too much again, and there are none of either kind where those would too.  Time over the general plan's, mean and worst of 8150 drawn decode
// and candidate calls of 0.7 MiB to 1.2 GiB, by the MiB read again and by all that the call reads (below 64 MiB / 64 to 256 / more):
//   units of 16:                             up to 32 0.54, 1.04 / 0.80, 1.05 / 0.84, 1.04;  32 to 56 0.57, 1.04 / 0.81, 1.22 / 0.90, 1.11;
//                                            56 to 112 0.60, 1.09 / 0.88, 1.32 / 0.93, 1.12;  112 to 200 0.63, 1.21 / 1.00, 1.78 / 1.00, 1.23;
//   units of 32, trees of at most 64 rows:   up to 56 0.81, 1.30 / 0.91, 1.28 / 0.89, 1.20;  56 to 112 0.79, 0.99 / 1.00, 1.32 / 0.99, 1.38;
//   trees of more, which are units of two
//   row tiles per wavefront otherwise:       up to 56 0.54, 1.05 / 0.77, 1.04 / 0.76;  56 to 112 0.60, 1.07 / 0.86, 1.16 / 0.83, 0.95;
//                                            112 to 200 0.63, 0.99 / 0.93, 1.47 / 0.94, 1.15.
// With 112 MiB for all trees 292 of 4745 calls with trees of at most 64 rows were slower than under the general plan by more than 3 % (the worst
// 1.38 times), now 133 (1.31), at the same mean (0.78).
constexpr int64_t kFewAgainBytes = (int64_t)56 << 20, kFewAgainWideBytes = (int64_t)112 << 20, kFewAgainNarrowBytes = (int64_t)56 << 20;
constexpr int64_t kFewSmallBytes = (int64_t)64 << 20;
constexpr int32_t kFewUnits = 1024;

// Which units of a decode plan are cut into slices (attn_split.hpp), and the launch's workgroups in order.  A unit's cost
// is the tiles a wavefront of it walks.  With T = total cost / shares, but at least kSliceMinTiles, units of more than T
// tiles become slices of about T; where no unit does, `out` stays empty and the launch has one workgroup per unit.
// Measured (us per call, uncut / 256 / 512 / 1024 shares; trees of two fork levels, 32 q heads):
//   bf16, 32 kv heads:  1 request 36 / 24 / 24 / 24,  4: 88 / 44 / 44 / 47,  16: 182 / 170 / 162 / 162,  32: 251 / 252 / 266 / 258
//   bf16, 8 kv heads:   1 request 41 / 22 / 22 / 22,  4: 98 / 67 / 70 / 70,  16: 136 / 96 / 97 / 96
//   one thread family of 32 k tokens, 8 kv heads: 106 / 58 / 59 / 63;  five candidates, 16 requests: 189 / 189 / 221 / 222
// Slices of 4, 2 and 1 tiles instead of kSliceMinTiles: 25, 32 and 32 against 22 us for one request with 8 kv heads.
// Slices are worth their states and their fold only where they shorten the longest walk by more than kSliceMinGain
// tiles (26 requests, 8 kv heads, units of 19 to 27 tiles: 46 us uncut, 49 us with every unit cut in two).  Their room is an
// eighth of the pool, at least 1 MiB and at most kSplitStateBytes; where it is short, T grows until the states fit (by a quarter
// at a time: a pass over the units each, nothing is built) or nothing is worth cutting any more.
constexpr int kSliceShares = 256;
constexpr int kSliceMinTiles = 6, kSliceMinGain = 16;
// Calls of few workgroups: shorter slices pay, since every wavefront folds a quarter of them, but only as long as there are no
// more workgroups than compute units (two on one share its 50 bytes per cycle).  Shares / least tiles / least gain, us per call:
//   256 / 6 / 16, 128 / 4 / 5, 192 / 4 / 5, 224 / 4 / 5: one request of 5 threads, 32 heads 9.7, 8.7, 8.4, 8.6, 8 heads 9.7, 8.6, 8.2, 8.5; two
//   requests 14.1, 12.1, 10.8, 11.0; four 18.7, 15.1, 17.8, 20.4; eight, 8 heads 19.4, 17.0, 16.3, 21.0; 32 k tokens, 8 heads 34.3, 32.4, 31.7,
//   32.8; three requests of 7 k to 11 k 116, 87, 90, 115; eight of 4 k on fp8, 8 heads 28.9, 28.4, 26.0, 29.4.
constexpr int kFewShares = 192, kFewMinTiles = 4, kFewMinGain = 5;
constexpr int32_t kFewWorkgroups = 256;
// fp32 pools: wavefronts are busy with products (a tile of d = 128 is 2048 cycles of them), so what a call takes is the largest sum
// of walks on one compute unit.  Tiles per slice are those whose estimate is least:
//   max(1.2 x longest slice, workgroups per compute unit, rounded up, x mean slice) + (3 + 0.45 x slices of the most cut unit)
// in tiles; a workgroup alone on its compute unit has nobody to fill its softmax (1.2), and a state to fold costs 0.45 tiles.
// Measured, us per call, by tiles per slice (workgroups): one request of 8 k tokens, 8 heads 3 to 4 (264) 33, 4 (256) 26.8, 6 (168) 25.7; of
// 4 k to 14 k, group 5 7 (448) 45, 13 (256) 38.7, 17 (192) 37.9; eight of 2 k to 5 k 17 (256) 31.7, 9 (512) 30.5; one of 14 k with 30 threads of
// four candidates 53 (256) 78, 35 (384) 60.8, 27 (512) 64.8; one of five threads, group 4 14 (16) 20.4, 4 (64) 13.2, 3 (80) 12.4; four of
// group 4 4 (220) 18.4, 3 (264) 22.8.
// The estimate knows units whose wavefronts leave one state of one row tile together.  Plans with shared lists, whose wavefronts leave one to two
// row tiles of state each, and calls of more than 512 units (kv heads counted) are cut by shares, as 16-bit pools cut theirs, into 512.  Time by
// the estimate over that by shares, mean and worst of 3000 drawn calls, by units:
//   without shared lists, up to 128 0.79, 1.17; 128 to 256 0.94, 1.25; 256 to 512 0.93, 1.23; 512 to 1024 1.00, 1.11; 1024 to 4096 1.01, 1.08;
//   with them, one row tile up to 512 0.93, 1.04, more 1.03, 1.17; two up to 512 0.97, 1.22, 512 to 1024 1.03, 1.33, more 1.02, 1.14.
// (With the estimate up to 4096 units for every plan 169 of the 3000 calls were slower by more than 3 % than with shares and the general plan, now 43.)
constexpr size_t kEstimatedUnits = 512;
constexpr int kSliceSharesF32 = 512;
int64_t tiles_per_slice_f32(const PlanHost& ph, const std::vector<int32_t>& units_of_cost, int64_t total, int n_kv) {
    const int32_t longest = (int32_t)units_of_cost.size() - 1;
    struct Kind {
        int32_t cost, units;
    };
    std::vector<Kind> kinds;
    for (int32_t c = longest; c >= 0; --c)
        if (units_of_cost[c] > 0) kinds.push_back(Kind{c, units_of_cost[c]});
    double best = 0.0;
    int32_t pick = longest;
    for (int32_t t = longest;; t = (int32_t)((int64_t)t * 4 / 5)) {
        int64_t n = (int64_t)ph.wgs.size();
        int32_t slice = 0, most = 1;
        for (const Kind& u : kinds) {
            if (u.cost <= t) {
                slice = std::max(slice, u.cost);
                break;
            }
            const int32_t k = std::min(64, (u.cost + t - 1) / t);
            n += (int64_t)(k - 1) * u.units, most = std::max(most, k), slice = std::max(slice, (u.cost + k - 1) / k);
        }
        const int64_t per_cu = (n * n_kv + 255) / 256;
        const double est = std::max(1.2 * slice, (double)per_cu * total / n) + (most > 1 ? 3.0 + 0.45 * most : 0.0);
        if (t == longest || est < best) best = est, pick = t;
        if (t <= 3) break;
    }
    return pick;
}
void cut_into_slices(const PlanHost& ph, const Shape& s, bool few, size_t state_bytes, std::vector<SplitBlock>& out, int32_t (&n_class)[3]) {
    out.clear();
    n_class[0] = n_class[1] = n_class[2] = 0;
    if (state_bytes == 0) return;
    auto cost = [](const WgDesc& wg) {
        return wg.n_coop + std::max(std::max(wg.w[0].n_tiles, wg.w[1].n_tiles), std::max(wg.w[2].n_tiles, wg.w[3].n_tiles));
    };
    // 16-row tiles of state that a slice of the unit leaves (the kernel for few units takes all of a call's as it takes the widest)
    const int at_least = few && ph.n_wg_class[1] > 0 ? 2 : 1;
    auto state_of = [at_least](const WgDesc& wg) { return ((wg.w[0].flags & kWaveSplit) ? 1 : 4) * std::max(at_least, wg.row_tiles & 255); };
    const size_t first = (size_t)ph.n_wg_class[0];  // (matrix units stay whole)
    int64_t total = 0;
    int longest = 0;
    for (size_t k = first; k < ph.wgs.size(); ++k) {
        const int c = cost(ph.wgs[k]);
        total += c;
        longest = std::max(longest, c);
    }
    few = few && (int64_t)ph.wgs.size() * s.n_kv <= kFewWorkgroups;
    const int64_t shares = few ? kFewShares : s.dtype == APAR_F32 ? kSliceSharesF32 : kSliceShares;
    int64_t tiles = std::max<int64_t>(few ? kFewMinTiles : kSliceMinTiles, (total * s.n_kv + shares - 1) / shares);
    int min_gain = few ? kFewMinGain : kSliceMinGain;
    if (s.dtype == APAR_F32 && ph.wgs.size() * s.n_kv <= kEstimatedUnits &&
        std::none_of(ph.wgs.begin(), ph.wgs.end(), [](const WgDesc& wg) { return wg.n_coop > 0; })) {
        std::vector<int32_t> units_of_cost((size_t)longest + 1, 0);
        for (const WgDesc& wg : ph.wgs) units_of_cost[cost(wg)] += 1;
        tiles = tiles_per_slice_f32(ph, units_of_cost, total, s.n_kv);
        min_gain = 0;
    }
    auto slices_of = [&](size_t k) { return k < first ? 1 : (int)std::min<int64_t>(64, (cost(ph.wgs[k]) + tiles - 1) / tiles); };
    const int64_t room = (int64_t)state_bytes / (s.n_kv * (int64_t)(s.d / 4 + 2) * 64 * (int64_t)sizeof(float));
    for (;; tiles += (tiles + 3) / 4) {
        if (longest <= tiles + min_gain) return;
        int64_t state = 0, blocks = 0, cut = 0;
        for (size_t k = first; k < ph.wgs.size(); ++k) {
            const int n = slices_of(k);
            blocks += n;
            if (n > 1) state += (int64_t)n * state_of(ph.wgs[k]), cut += 1;
        }
        if (state <= room && cut * s.n_kv <= kSplitMaxCut && (!few || blocks * s.n_kv <= kFewWorkgroups)) break;
    }
    n_class[0] = (int32_t)first;
    int32_t state = 0, n_cut = 0;
    for (size_t k = 0; k < ph.wgs.size(); ++k) {
        const WgDesc& wg = ph.wgs[k];
        const int n = slices_of(k);
        for (int j = 0; j < n; ++j) out.push_back(SplitBlock{(int32_t)k, j | n << 16, state, n_cut});
        if (k >= first) n_class[(wg.row_tiles & 255) == 2 ? 1 : 2] += n;
        if (n > 1) {
            state += n * state_of(wg);
            n_cut += 1;
        }
    }
}

// Lays a small plan's tables out for the kernels' arguments: no upload, no staging slot and no event.  Only where nothing
// is left to merge (the merge kernel reads staged tables).  Measured per call: one request of five threads, 32 heads
// 22.5 -> 15.6 us, three threads on an fp32 pool 16.7 -> 9.4 us, a whole response (prompt, 16 steps of five threads) 435 -> 374 us.
// pack: the launcher packs them (units of a call of few units).
bool inline_plan(apar_pool* p, const PlanHost& ph, bool pack) {
    if (ph.any_partial || ph.n_wg_class[0] > 0) return false;
    const size_t n_blocks = p->split_blocks.empty() ? ph.wgs.size() : p->split_blocks.size();
    const size_t words = ph.wgs.size() * (sizeof(WgDesc) / 4) + n_blocks * (sizeof(SplitBlock) / 4) + ph.tiles.size() * (sizeof(TileRef) / 4) +
                         ph.dfs_threads.size();
    if ((pack ? few_packed_words(ph.wgs.size(), n_blocks, ph.tiles.size(), ph.dfs_threads.size()) : words) > (size_t)kPlanInlineWords) return false;
    p->inline_words.resize(words);
    char* base = (char*)p->inline_words.data();
    size_t at = 0;
    auto put = [&](int k, const void* from, size_t bytes) {
        p->inline_ofs[k] = at;
        memcpy(base + at, from, bytes);
        at += bytes;
    };
    put(0, ph.wgs.data(), ph.wgs.size() * sizeof(WgDesc));
    if (p->split_blocks.empty()) {  // units as they are
        p->inline_ofs[3] = at;
        for (size_t k = 0; k < n_blocks; ++k) {
            const SplitBlock b{(int32_t)k, 1 << 16, 0, 0};
            memcpy(base + at, &b, sizeof b);
            at += sizeof b;
        }
    } else {
        put(3, p->split_blocks.data(), n_blocks * sizeof(SplitBlock));
    }
    put(1, ph.tiles.data(), ph.tiles.size() * sizeof(TileRef));
    put(2, ph.dfs_threads.data(), ph.dfs_threads.size() * sizeof(int32_t));
    return true;
}

// What an open tile costs a wavefront of the 16-bit kernels, in full ones, where a list is cut four ways: its V half take a turn through
// LDS, and on fp8 pools it is twice the bytes.  On fp32 pools every tile is alike.  Counted as one, two and three, us per call: one request
// of five threads, 32 heads 9.4 / 8.8 / 8.8, four requests 17.6 / 18.5 / 17.7, 60 requests, 4 heads 22.0 / 21.3 / 21.1, twelve short ones, 8 heads 12.6 /
// 12.3 / 12.0, 64 requests, 32 heads 214.8 / 213.4 / 213.9; fp8 one request 10.0 / 9.4 / 9.1, three short ones 9.5 / 8.7 / 8.5, 64 requests, 8 heads 41.5 / 41.8 / 41.8.
constexpr int kOpenTileCost = 2;

// fixed: the plan and the partial results go to the device's static workspace, nothing is allocated, no
// stream or event is created and profiling is off for the call.
int decode_common(apar_pool* p, const void* q, const void* cand_k, const void* cand_v, const uint8_t* mask,
                  int n_cand, const apar_thread* ids, int n, void* out, void* stream, bool spec, bool fixed = false) {
    if (!p || n < 0) return APAR_ERR_INVALID_ARG;
    if (fixed && (p->dry_run || !p->fixed_dev || !p->fixed_host)) return APAR_ERR_INVALID_ARG;
    if (n == 0) return APAR_OK;
    if (!ids) return APAR_ERR_INVALID_ARG;
    if (spec && (n_cand < 1 || n_cand > 8)) return APAR_ERR_INVALID_ARG;
    if (p->dry_run) {
        if (q || out || cand_k || cand_v || mask) return APAR_ERR_INVALID_ARG;
    } else {
        if (!q || !out) return APAR_ERR_INVALID_ARG;
        if (spec && (!cand_k || !cand_v || !mask)) return APAR_ERR_INVALID_ARG;
    }
    const auto t0 = std::chrono::steady_clock::now();
    p->wait_in_call_ms = 0.0;

    p->views.resize(n);
    for (int i = 0; i < n; ++i) {
        if (i + 16 < n && ids[i + 16] >= 0 && (size_t)ids[i + 16] < p->threads.size()) __builtin_prefetch(&p->threads[ids[i + 16]]);
        Thread* t = live_thread(p, ids[i]);
        if (!t) return APAR_ERR_INVALID_THREAD;
        if (t->len == 0) return APAR_ERR_INVALID_ARG;
        p->views[i] = PlanThreadView{t->table.data(), (int32_t)t->table.size(), t->len};
    }
    PlanHost& ph = p->plan;
    PlanParams prm;
    prm.rows_per_thread = n_cand * p->shape.group;
    prm.max_unit_tiles = p->max_unit_tiles;
    prm.allow_direct = true;
    prm.fuse = true;
    prm.matrix_min_rows = p->has_matrix_units() ? p->matrix_min_rows : 0;
    prm.matrix_min_blocks = p->matrix_min_blocks;
    prm.inline_shared = p->inline_shared;
    prm.open_cost = p->shape.dtype == APAR_F32 ? 1 : kOpenTileCost;
    prm.few_units = p->planning_set ? 0 : kFewUnits / p->shape.n_kv;
    // (the fp32 kernel's wavefronts read shared lists one by one: units of 16 rows read nothing more often)
    const int64_t tile_read = p->shape.n_kv * (p->shape.fp8_sealed ? 4096 : 8192);
    prm.few_row_tiles = p->shape.dtype == APAR_F32 ? 1 : 2;
    prm.few_again = p->shape.dtype == APAR_F32 ? INT32_MAX : (int32_t)(kFewAgainBytes / tile_read);
    prm.few_again_wide = (int32_t)(kFewAgainWideBytes / tile_read);
    prm.few_again_narrow = (int32_t)(kFewAgainNarrowBytes / tile_read);
    prm.few_small = (int32_t)(kFewSmallBytes / tile_read);
    prm.few_open_cost = p->shape.fp8_sealed ? 2 : 1;  // (twice the bytes of a full one)
    // Decode calls of a loop list the same threads step after step - each a few rows longer, a few replaced
    // by a thread forked from them - and the plan of the previous call then only needs its tails brought up
    // to date.  A table never changes before its last block, and a thread forked since the previous call
    // started from a copy of its parent's table as it was then or later, so "position by position the same
    // thread or one forked from it since" is all that has to hold for patch_plan to apply.
    bool carried = false;
    if (p->plan_reuse && ph.reusable && (size_t)n == p->plan_ids.size() && prm == p->plan_prm) {
        bool same = true;
        for (int i = 0; i < n && same; ++i) {
            int32_t t = ids[i];
            while (t != p->plan_ids[i] && t >= 0 && (size_t)t >= p->plan_threads_then) t = p->threads[t].forked_from;
            same = t == p->plan_ids[i];
        }
        carried = same && patch_plan(p->views.data(), n, p->cow_copies == p->plan_copies_then, ph);
    }
    int rc = carried ? APAR_OK : build_plan(p->views.data(), n, p->ref.data(), p->seg_of.data(), prm, ph);
    if (rc != APAR_OK) {
        ph.reusable = false;
        return rc;
    }
    p->plan_ids.assign(ids, ids + n);
    p->plan_prm = prm;
    p->plan_threads_then = p->threads.size();
    p->plan_copies_then = p->cow_copies;
    (carried ? p->n_plans_carried : p->n_plans_built) += 1;
    const int64_t e = p->shape.dtype == APAR_F32 ? 4 : 2;
    apar_plan_info info{};
    info.n_threads = n;
    info.n_segments = ph.n_segments;
    info.n_units = (int64_t)ph.wgs.size() * p->shape.n_kv;
    info.n_partial_rows = ph.n_partial_rows;
    info.unique_blocks = ph.unique_blocks;
    info.unique_tokens = ph.unique_tokens;
    info.path_tokens = ph.path_tokens;
    info.algorithmic_bytes = ph.unique_tokens * 2 * p->shape.n_kv * p->shape.d * e +
                             2 * (int64_t)n * n_cand * p->shape.n_q * p->shape.d * e;
    if (p->shape.fp8_sealed)  // full blocks: one byte per element and two scales per (block, kv head)
        info.algorithmic_bytes -= ph.full_blocks * ((int64_t)kBlockTokens * p->shape.n_kv * p->shape.d * 2 - 8 * p->shape.n_kv);
    if (spec) info.algorithmic_bytes += 2 * (int64_t)n * n_cand * p->shape.n_kv * p->shape.d * e;
    p->plan_geom[0] = prm.rows_per_thread;
    p->plan_geom[2] = (prm.rows_per_thread + 15) / 16;
    p->plan_geom[1] = (prm.rows_per_thread + p->plan_geom[2] - 1) / p->plan_geom[2];
    if (p->dry_run) {
        p->last_plan = info;
        return APAR_OK;
    }
    DeviceGuard guard(p->device);
    hipStream_t st = (hipStream_t)stream;

    const bool few = ph.few_row_tiles > 0 && p->shape.dtype != APAR_F32;  // (fp32 pools have one kernel for all units)
    if (!carried) cut_into_slices(ph, p->shape, few, p->split_bytes, p->split_blocks, p->n_split_class);  // (a carried plan keeps its cut)
    // stage the tables in one copy
    size_t ofs[7];
    ofs[0] = 0;
    ofs[1] = align_up(ofs[0] + ph.wgs.size() * sizeof(WgDesc), 256);
    ofs[2] = align_up(ofs[1] + ph.tiles.size() * sizeof(TileRef), 256);
    ofs[3] = align_up(ofs[2] + ph.dfs_threads.size() * 4, 256);
    ofs[4] = align_up(ofs[3] + ph.path_ofs.size() * 4, 256);
    ofs[5] = align_up(ofs[4] + ph.path_ids.size() * 4, 256);
    ofs[6] = align_up(ofs[5] + p->split_blocks.size() * sizeof(SplitBlock), 256);
    const size_t staged = ofs[6];
    bool cut = !p->split_blocks.empty();
    const size_t slots = (size_t)ph.n_partial_rows * n_cand * p->shape.n_q;
    StageSlot* s = nullptr;
    char *host = nullptr, *dev = nullptr;
    size_t fixed_bytes = 0;
    PartialBuf part = p->part;
    if (p->resident_behind) p->resident = nullptr;
    p->resident_behind = false;
    const bool pack = few && p->cfg.num_blocks <= kFewPackedBlocks;
    const bool inlined = !fixed && inline_plan(p, ph, pack);
    // a carried-over plan whose tables are still on the device from the previous call: only the words that
    // changed are sent, and written in place once the previous call's kernels are through (one launch, as a copy of the whole
    // tables is: a step of 64 requests, 32 heads, one row per thread and call 0.386 -> 0.380 ms; a serving loop with at most 64
    // requests 1.45 -> 1.49 M output tokens per second)
    const bool in_place = carried && !fixed && !inlined && p->resident && p->resident_bytes == staged;
    if (!in_place) p->resident = nullptr;
    if (in_place) {
        p->resident_behind = true;
        StageSlot* res = p->resident;
        if (res->pending) HIP_TRY(hipStreamWaitEvent(st, res->ev, 0));  // (a no-op on the stream of the previous call)
        const size_t n_pairs = ph.dirty_wg_words.size() + ph.dirty_tile_words.size();
        if (n_pairs > 0) {
            StageSlot* ps = nullptr;
            if ((rc = acquire_stage(p, n_pairs * 2 * sizeof(int32_t), &ps)) != APAR_OK) return rc;
            int32_t* pairs = (int32_t*)ps->host;
            const int32_t* wg_words = (const int32_t*)ph.wgs.data();
            const int32_t* tile_words = (const int32_t*)ph.tiles.data();
            const int32_t wg_base = (int32_t)(ofs[0] / 4), tile_base = (int32_t)(ofs[1] / 4);
            for (int32_t w : ph.dirty_wg_words) *pairs++ = wg_base + w, *pairs++ = wg_words[w];
            for (int32_t w : ph.dirty_tile_words) *pairs++ = tile_base + w, *pairs++ = tile_words[w];
            HIP_TRY(launch_scatter_words((int32_t*)res->dev, (const int32_t*)ps->host, (int)n_pairs, st));
            HIP_TRY(hipEventRecord(ps->ev, st));
            ps->pending = true;
        }
        p->resident_behind = false;
        s = res;
        dev = res->dev;
    } else if (fixed) {
        // the workspace has a fixed size: a plan or a set of partial results beyond it is refused
        const size_t slot_bytes = (size_t)(p->shape.d + 2) * sizeof(float);
        const size_t cap_slots = kFixedPartBytes / slot_bytes;
        if (ofs[5] > kFixedPlanBytes || slots > cap_slots) return APAR_ERR_WORKSPACE_LIMIT;
        if (p->fixed_pending) {  // the previous call's upload may still be reading the pinned buffer
            HIP_TRY(hipEventSynchronize(p->fixed_up));
            p->fixed_pending = false;
        }
        host = p->fixed_host;
        dev = p->fixed_dev;
        part.o = (float*)(p->fixed_dev + kFixedPlanBytes);
        part.ml = part.o + cap_slots * p->shape.d;
        cut = cut && staged <= kFixedPlanBytes;
        fixed_bytes = cut ? staged : ofs[5];
    } else if (!inlined) {
        if ((rc = acquire_stage(p, staged, &s)) != APAR_OK) return rc;
        host = s->host;
        dev = s->dev;
    }
    if (!in_place && !inlined) {
        memcpy(host + ofs[0], ph.wgs.data(), ph.wgs.size() * sizeof(WgDesc));
        memcpy(host + ofs[1], ph.tiles.data(), ph.tiles.size() * sizeof(TileRef));
        memcpy(host + ofs[2], ph.dfs_threads.data(), ph.dfs_threads.size() * 4);
        memcpy(host + ofs[3], ph.path_ofs.data(), ph.path_ofs.size() * 4);
        if (!ph.path_ids.empty()) memcpy(host + ofs[4], ph.path_ids.data(), ph.path_ids.size() * 4);
        if (cut) memcpy(host + ofs[5], p->split_blocks.data(), p->split_blocks.size() * sizeof(SplitBlock));
    }

    // partial-result buffer
    if (!fixed && slots > p->part_slots_cap) {
        HIP_TRY(hipDeviceSynchronize());
        if (p->part.o) HIP_TRY(hipFree(p->part.o));
        if (p->part.ml) HIP_TRY(hipFree(p->part.ml));
        p->part = PartialBuf{};
        p->part_slots_cap = 0;
        const size_t cap = slots + slots / 4 + 1024;
        HIP_TRY(hipMalloc((void**)&p->part.o, cap * p->shape.d * sizeof(float)));
        HIP_TRY(hipMalloc((void**)&p->part.ml, cap * 2 * sizeof(float)));
        p->part_slots_cap = cap;
        part = p->part;
    }

    if (in_place || inlined) {
        // (already there, or on its way with the kernels)
    } else if (fixed) {
        HIP_TRY(copy_staged(dev, host, fixed_bytes, st));
        HIP_TRY(hipEventRecord(p->fixed_up, st));
        p->fixed_pending = true;
    } else if ((rc = upload(p, s, staged, st)) != APAR_OK) {
        return rc;
    }
    part.stream = slots * (size_t)(p->shape.d + 2) * sizeof(float) > kStreamPartialBytes;
    PlanDev pd{};
    pd.wgs = (const WgDesc*)(dev + ofs[0]);
    pd.tiles = (const TileRef*)(dev + ofs[1]);
    pd.dfs_threads = (const int32_t*)(dev + ofs[2]);
    pd.path_ofs = (const int32_t*)(dev + ofs[3]);
    pd.path_ids = (const int32_t*)(dev + ofs[4]);
    pd.n_wg = (int32_t)ph.wgs.size();
    for (int k = 0; k < 3; ++k) pd.n_wg_class[k] = ph.n_wg_class[k];
    if (pd.n_wg_class[0] + pd.n_wg_class[1] + pd.n_wg_class[2] != pd.n_wg) return APAR_ERR_INVALID_ARG;
    pd.n_threads = n;
    pd.rows_per_thread = p->plan_geom[0];
    pd.rows_per_slice = p->plan_geom[1];
    pd.n_slices = p->plan_geom[2];
    if (cut) {
        pd.split.blocks = (const SplitBlock*)(dev + ofs[5]);
        for (int k = 0; k < 3; ++k) pd.split.n_blocks_class[k] = p->n_split_class[k];
    }
    pd.split.arrived = (int32_t*)p->split_dev;  // (no room: nothing is cut and nothing reads either)
    pd.split.state = p->split_dev ? (float*)(p->split_dev + kSplitCounterBytes) : nullptr;

    pd.few = few ? (inlined && pack ? 2 : 1) : 0;

    if (inlined) {
        pd.wgs = (const WgDesc*)p->inline_ofs[0];
        pd.tiles = (const TileRef*)p->inline_ofs[1];
        pd.dfs_threads = (const int32_t*)p->inline_ofs[2];
        pd.path_ofs = pd.path_ids = nullptr;  // (nothing to merge)
        pd.split.blocks = (const SplitBlock*)p->inline_ofs[3];
        for (int k = 0; k < 3; ++k) pd.split.n_blocks_class[k] = cut ? p->n_split_class[k] : ph.n_wg_class[k];
        pd.inline_words = p->inline_words.data();
        pd.n_inline_words = (int32_t)p->inline_words.size();
    }

    EventPair ev;
    const bool profiling = p->profiling && !fixed;
    if (profiling) {
        if ((rc = new_event(p, &ev.a)) != APAR_OK || (rc = new_event(p, &ev.b)) != APAR_OK ||
            (rc = new_event(p, &ev.c)) != APAR_OK)
            return rc;
        HIP_TRY(hipEventRecord(ev.a, st));
    }
    if (cut && !p->split_clear) {
        HIP_TRY(launch_clear_words((int32_t*)p->split_dev, (int)(kSplitCounterBytes / sizeof(int32_t)), st));
        // (a call that is being captured runs its own clear when it is replayed; nothing is cleared before that)
        hipStreamCaptureStatus capture = hipStreamCaptureStatusNone;
        if (hipStreamIsCapturing(st, &capture) != hipSuccess) (void)hipGetLastError();
        else p->split_clear = capture == hipStreamCaptureStatusNone;
    }
    HIP_TRY(launch_attention_partial(p->shape, p->kv, q, pd, n_cand, part, cand_k, cand_v, mask, out, st));
    if (profiling) HIP_TRY(hipEventRecord(ev.b, st));
    if (ph.any_partial)
        HIP_TRY(launch_merge(p->shape, pd, part, q, cand_k, cand_v, mask, n_cand, out, st));
    if (profiling) {
        HIP_TRY(hipEventRecord(ev.c, st));
        p->decode_events.push_back(ev);
        p->n_decode_calls += 1;
    }
    if (s) {
        HIP_TRY(hipEventRecord(s->ev, st));
        s->pending = true;
        p->resident = s;
        p->resident_bytes = staged;
    }
    p->last_plan = info;
    if (profiling)
        p->plan_host_ms += std::chrono::duration<double, std::milli>(std::chrono::steady_clock::now() - t0).count() -
                           p->wait_in_call_ms;
    return APAR_OK;
}

// Whether a prefill call on a bf16 or fp8 pool goes to the 32x32 kernel by itself.  That kernel gives a workgroup up to 128
// query rows (tokens x q heads of a kv group) of one thread; a row-tile workgroup with one row tile per wavefront holds 64.
//  - Threads of more than 64 rows are faster there, the others mostly on the row tiles: what decides is the rows that the
//    workgroups of either kind walk, so that one long prompt does not take hundreds of short threads with it.
//    Measured (us, row tiles / matrix kernel; 362 threads, six to a shared prefix, walks around 400): bf16 group 2, 62 and 78 rows
//    164 / 184, 258 / 202; group 4, 64 and 80 rows 90 / 94, 134 / 99; fp8 pools group 1, 59 and 69 rows 305 / 345, 477 / 375, group 4,
//    64 and 80 rows 88 / 98, 137 / 103, group 8, 112 rows 82 / 66; walks around 1050, group 4: bf16 181 / 184, 282 / 203, fp8
//    170 / 184, 277 / 204.  360 threads of one row and walks of 300 beside a prompt of 2000, group 8: bf16 88 / 71, fp8 91 / 75.
//    Where the line lies on the slower side: group 16, 64 rows 48 / 36; fp8 group 8, 48 rows 124 / 110; one row and walks of 900
//    beside a prompt of 2000, group 4 179 / 154, group 1 556 / 477; 8 to 40 requests of 48 rows, group 4, by 6 to 9 %.
//  - bf16 pools: from 32 rows per workgroup on, a large call (kMatrixPrefillWalked rows walked by all its workgroups, kv
//    heads counted) goes there all the same, which is even or a little faster: group 1, 48 rows, 362 threads of walks around 400,
//    700, 1050 (4.6, 8, 12 M) 325 / 343, 492 / 484, 693 / 672; group 4, 48 rows, 891 threads (2.9, 5, 7.5 M) 197 / 218, 307 / 320,
//    440 / 437, group 1, 891 threads, walks around 700 1224 / 1172; and calls whose query tokens attend to kMatrixPrefillMeanWalk rows
//    on average go there (group 1, one token each, 362 threads, around 1100 rows: 499 / 523 where six share a prefix, 1080 / 1077 where
//    nobody does).  fp8 pools: neither (362 threads, group 4, around 1050 rows, 32 and 64 rows 170 / 156, 170 / 184).
constexpr int64_t kMatrixPrefillRows = 64, kMatrixPrefillMinRows = 32;
constexpr int64_t kMatrixPrefillWalked = 4500000;
constexpr int64_t kMatrixPrefillMeanWalk = 1024;
bool prefill_on_matrix(const Shape& s, const std::vector<PrefillThreadView>& views, int64_t rows, int64_t attended) {
    const int64_t chunk = 128 / s.group;
    int64_t wgs = 0, wide = 0, narrow = 0;
    for (const PrefillThreadView& t : views) {
        const int64_t w = (t.m + chunk - 1) / chunk;  // workgroups; each walks to its last token
        wgs += w;
        ((int64_t)t.m * s.group > kMatrixPrefillRows ? wide : narrow) += w * (t.len - t.m) + chunk * (w - 1) * w / 2 + t.m;
    }
    if (wide >= narrow) return true;
    if (s.fp8_sealed) return false;
    return attended >= kMatrixPrefillMeanWalk * rows ||
           (rows * s.group >= kMatrixPrefillMinRows * wgs && (wide + narrow) * s.n_kv >= kMatrixPrefillWalked);
}

// bf16 pools: the matrix-core prefill kernel.  One workgroup per (thread, chunk of 128 / group query tokens);
// the threads' block tables are staged next to the workgroup descriptors.
int prefill_bf16(apar_pool* p, const std::vector<PrefillThreadView>& views, int64_t rows, int64_t attended,
                 const void* q, void* out, void* stream, std::chrono::steady_clock::time_point t0) {
    const int group = p->shape.group;
    if (group < 1 || group > 16 || 16 % group != 0) return APAR_ERR_UNSUPPORTED;
    const int chunk = 128 / group;
    std::vector<PrefillWg>& wgs = p->prefill_wgs;
    std::vector<int32_t>& tables = p->prefill_tables;
    wgs.clear();
    tables.clear();
    for (const PrefillThreadView& t : views) {
        if (t.len > INT32_MAX / 2 || tables.size() + (size_t)t.n_blocks > (size_t)INT32_MAX / 2) return APAR_ERR_UNSUPPORTED;
        const int32_t table_ofs = (int32_t)tables.size();
        tables.insert(tables.end(), t.table, t.table + t.n_blocks);
        for (int64_t r0 = 0; r0 < t.m; r0 += chunk) {
            PrefillWg w{};
            w.table_ofs = table_ofs;
            w.q_row0 = (int32_t)(t.q_base + r0);
            w.p0 = (int32_t)(t.len - t.m + r0);
            w.n_tok = (int32_t)std::min<int64_t>(chunk, t.m - r0);
            w.len = (int32_t)t.len;
            wgs.push_back(w);
        }
    }
    // Workgroups of one tree (same first block) stay together, in the caller's order, so that the threads of a
    // tree walk their common prefix at about the same time and find it in the L2 of the XCD that serves their
    // kv head; trees with the longest walk go first so that the launch does not end on a long one.
    {
        std::unordered_map<int32_t, int32_t> longest;  // first block of a tree -> its longest walk
        for (const PrefillWg& w : wgs) {
            int32_t& e = longest[tables[w.table_ofs]];
            e = std::max(e, w.p0 + w.n_tok);
        }
        std::vector<std::pair<uint64_t, PrefillWg>> keyed;
        keyed.reserve(wgs.size());
        for (const PrefillWg& w : wgs) {
            const int32_t root = tables[w.table_ofs];
            keyed.emplace_back(((uint64_t)(uint32_t)(INT32_MAX - longest[root]) << 32) | (uint32_t)root, w);
        }
        std::stable_sort(keyed.begin(), keyed.end(),
                         [](const std::pair<uint64_t, PrefillWg>& a, const std::pair<uint64_t, PrefillWg>& b) {
                             return a.first < b.first;
                         });
        for (size_t i = 0; i < wgs.size(); ++i) wgs[i] = keyed[i].second;
    }
    apar_plan_info info{};
    info.n_threads = (int64_t)views.size();
    info.n_units = (int64_t)wgs.size() * p->shape.n_kv;
    info.path_tokens = attended;
    info.algorithmic_bytes = 2 * rows * p->shape.n_q * p->shape.d * 2;
    p->last_plan = info;
    DeviceGuard guard(p->device);
    hipStream_t st = (hipStream_t)stream;
    const size_t wg_bytes = align_up(wgs.size() * sizeof(PrefillWg), 256);
    const size_t table_bytes = tables.size() * sizeof(int32_t);
    StageSlot* s = nullptr;
    int rc = acquire_stage(p, wg_bytes + table_bytes, &s);
    if (rc != APAR_OK) return rc;
    memcpy(s->host, wgs.data(), wgs.size() * sizeof(PrefillWg));
    memcpy(s->host + wg_bytes, tables.data(), table_bytes);
    if ((rc = upload(p, s, wg_bytes + table_bytes, st)) != APAR_OK) return rc;
    EventPair ev;
    if (p->profiling) {
        if ((rc = new_event(p, &ev.a)) != APAR_OK || (rc = new_event(p, &ev.b)) != APAR_OK ||
            (rc = new_event(p, &ev.c)) != APAR_OK)
            return rc;
        HIP_TRY(hipEventRecord(ev.a, st));
    }
    HIP_TRY(launch_prefill_bf16(p->shape, p->kv, q, (const PrefillWg*)s->dev, (const int32_t*)(s->dev + wg_bytes),
                                (int)wgs.size(), out, st));
    if (p->profiling) {
        HIP_TRY(hipEventRecord(ev.b, st));
        HIP_TRY(hipEventRecord(ev.c, st));
        p->decode_events.push_back(ev);
        p->n_decode_calls += 1;
    }
    HIP_TRY(hipEventRecord(s->ev, st));
    s->pending = true;
    if (p->profiling)
        p->plan_host_ms += std::chrono::duration<double, std::milli>(std::chrono::steady_clock::now() - t0).count() -
                           p->wait_in_call_ms;
    return APAR_OK;
}

int prefill_common(apar_pool* p, const void* q, const apar_thread* ids, const int32_t* m, int n, void* out,
                   void* stream) {
    if (!p || n < 0) return APAR_ERR_INVALID_ARG;
    if (n == 0) return APAR_OK;
    if (!ids || !m) return APAR_ERR_INVALID_ARG;
    if (p->dry_run ? (q || out) : (!q || !out)) return APAR_ERR_INVALID_ARG;
    const auto t0 = std::chrono::steady_clock::now();
    p->wait_in_call_ms = 0.0;
    std::vector<PrefillThreadView>& views = p->prefill_views;
    views.resize(n);
    int64_t rows = 0, attended = 0;
    for (int i = 0; i < n; ++i) {
        Thread* t = live_thread(p, ids[i]);
        if (!t) return APAR_ERR_INVALID_THREAD;
        if (m[i] < 1 || m[i] > t->len) return APAR_ERR_INVALID_ARG;
        views[i] = PrefillThreadView{t->table.data(), (int32_t)t->table.size(), t->len, m[i], rows};
        rows += m[i];
        attended += (int64_t)m[i] * (t->len - m[i]) + (int64_t)m[i] * (m[i] + 1) / 2;
    }
    if (rows > INT32_MAX / 2) return APAR_ERR_UNSUPPORTED;
    PlanHost& ph = p->plan;
    int rc = APAR_OK;
    p->last_prefill_kernel = APAR_PREFILL_ROW_TILES;
    // (an fp8 pool takes the matrix kernel by AUTO only)
    if (!p->dry_run && p->shape.dtype == APAR_BF16 && 16 % p->shape.group == 0 &&
        ((p->prefill_kernel == APAR_PREFILL_MATRIX && !p->shape.fp8_sealed) ||
         (p->prefill_kernel == APAR_PREFILL_AUTO && prefill_on_matrix(p->shape, views, rows, attended)))) {
        p->last_prefill_kernel = APAR_PREFILL_MATRIX;
        return prefill_bf16(p, views, rows, attended, q, out, stream, t0);
    }
    rc = build_prefill_plan(views.data(), n, p->shape.group, ph);
    if (rc != APAR_OK) return rc;
    apar_plan_info info{};
    info.n_threads = n;
    info.n_units = (int64_t)ph.wgs.size() * p->shape.n_kv;
    info.path_tokens = attended;  // (query token, attended row) pairs
    const int64_t e = p->shape.dtype == APAR_F32 ? 4 : 2;
    info.algorithmic_bytes = 2 * rows * p->shape.n_q * p->shape.d * e;  // queries in, outputs out; K,V reads depend on caching
    p->plan_geom[0] = p->plan_geom[1] = p->shape.group;
    p->plan_geom[2] = 1;
    p->last_plan = info;
    if (p->dry_run) return APAR_OK;
    DeviceGuard guard(p->device);
    hipStream_t st = (hipStream_t)stream;
    const size_t wg_bytes = align_up(ph.wgs.size() * sizeof(WgDesc), 256);
    const size_t tile_bytes = ph.tiles.size() * sizeof(TileRef);
    StageSlot* s = nullptr;
    if ((rc = acquire_stage(p, wg_bytes + tile_bytes, &s)) != APAR_OK) return rc;
    memcpy(s->host, ph.wgs.data(), ph.wgs.size() * sizeof(WgDesc));
    if (tile_bytes) memcpy(s->host + wg_bytes, ph.tiles.data(), tile_bytes);
    if ((rc = upload(p, s, wg_bytes + tile_bytes, st)) != APAR_OK) return rc;
    PlanDev pd{};
    pd.wgs = (const WgDesc*)s->dev;
    pd.tiles = (const TileRef*)(s->dev + wg_bytes);
    pd.dfs_threads = nullptr;  // a row group is a query token, numbered as q_dev's rows are
    pd.path_ofs = pd.path_ids = nullptr;
    pd.n_wg = (int32_t)ph.wgs.size();
    for (int k = 0; k < 3; ++k) pd.n_wg_class[k] = ph.n_wg_class[k];
    pd.n_threads = (int32_t)rows;
    pd.rows_per_thread = pd.rows_per_slice = p->shape.group;
    pd.n_slices = 1;
    EventPair ev;
    if (p->profiling) {
        if ((rc = new_event(p, &ev.a)) != APAR_OK || (rc = new_event(p, &ev.b)) != APAR_OK ||
            (rc = new_event(p, &ev.c)) != APAR_OK)
            return rc;
        HIP_TRY(hipEventRecord(ev.a, st));
    }
    HIP_TRY(launch_attention_partial(p->shape, p->kv, q, pd, 1, p->part, nullptr, nullptr, nullptr, out, st));
    if (p->profiling) {
        HIP_TRY(hipEventRecord(ev.b, st));
        HIP_TRY(hipEventRecord(ev.c, st));
        p->decode_events.push_back(ev);
        p->n_decode_calls += 1;
    }
    HIP_TRY(hipEventRecord(s->ev, st));
    s->pending = true;
    if (p->profiling)
        p->plan_host_ms += std::chrono::duration<double, std::milli>(std::chrono::steady_clock::now() - t0).count() -
                           p->wait_in_call_ms;
    return APAR_OK;
}

}  // namespace

// ===========================================================================
// C ABI
// ===========================================================================
extern "C" {

int apar_pool_create(const apar_pool_config* cfg, void* kv_dev, size_t kv_bytes, apar_pool** out) {
    if (!cfg || !out) return APAR_ERR_INVALID_ARG;
    if (!kv_dev && kv_bytes != 0) return APAR_ERR_INVALID_ARG;
    *out = nullptr;
    if (cfg->block_size != kBlockTokens) return APAR_ERR_INVALID_ARG;
    if (cfg->n_q_heads < 1 || cfg->n_kv_heads < 1 || cfg->n_q_heads % cfg->n_kv_heads) return APAR_ERR_INVALID_ARG;
    if (cfg->num_blocks < 1 || cfg->num_blocks > kMaxPoolBlocks || cfg->max_threads < 1)
        return APAR_ERR_INVALID_ARG;
    if (cfg->dtype != APAR_F32 && cfg->dtype != APAR_BF16 && cfg->dtype != APAR_BF16_FP8KV) return APAR_ERR_INVALID_ARG;
    if (!(cfg->softmax_scale >= 0.0f) || !std::isfinite(cfg->softmax_scale)) return APAR_ERR_INVALID_ARG;
    if (cfg->dtype != APAR_F32 && cfg->head_dim != 128) return APAR_ERR_UNSUPPORTED;
    if (cfg->dtype == APAR_F32 && cfg->head_dim != 64 && cfg->head_dim != 128) return APAR_ERR_UNSUPPORTED;
    if (cfg->n_q_heads / cfg->n_kv_heads > 16) return APAR_ERR_UNSUPPORTED;
    const int64_t e = cfg->dtype == APAR_F32 ? 4 : 2;
    const int64_t tile = 2 * (int64_t)kBlockTokens * cfg->head_dim * e;
    const int64_t block = tile * cfg->n_kv_heads;
    if (kv_dev && ((uint64_t)kv_bytes < (uint64_t)(block * cfg->num_blocks) || ((uintptr_t)kv_dev & 255)))
        return APAR_ERR_INVALID_ARG;

    apar_pool* p = new (std::nothrow) apar_pool();
    if (!p) return APAR_ERR_INVALID_ARG;
    p->cfg = *cfg;
    p->kv = (char*)kv_dev;
    p->dry_run = kv_dev == nullptr;
    if (!p->dry_run) {
        if (!hip_ok(hipGetDevice(&p->device), "hipGetDevice")) {
            delete p;
            return APAR_ERR_HIP;
        }
        hipPointerAttribute_t attr;
        if (hipPointerGetAttributes(&attr, kv_dev) == hipSuccess) p->device = attr.device;
        else (void)hipGetLastError();
        DeviceGuard guard(p->device);
        const int rc = set_up_workspace(p, (size_t)(block * cfg->num_blocks));
        if (rc != APAR_OK) {
            release_workspace(p);
            delete p;
            return rc;
        }
    }
    const float scale = cfg->softmax_scale > 0.0f ? cfg->softmax_scale : 1.0f / std::sqrt((float)cfg->head_dim);
    p->shape.n_q = cfg->n_q_heads;
    p->shape.n_kv = cfg->n_kv_heads;
    p->shape.d = cfg->head_dim;
    p->shape.group = cfg->n_q_heads / cfg->n_kv_heads;
    p->shape.dtype = cfg->dtype == APAR_F32 ? APAR_F32 : APAR_BF16;
    p->shape.fp8_sealed = cfg->dtype == APAR_BF16_FP8KV ? 1 : 0;
    p->shape.scale_log2e = scale * 1.4426950408889634f;
    p->shape.tile_bytes = tile;
    p->shape.block_bytes = block;
    p->ref.assign(cfg->num_blocks, 0);
    p->free_stack.resize(cfg->num_blocks);
    for (int64_t i = 0; i < cfg->num_blocks; ++i) p->free_stack[i] = (int32_t)(cfg->num_blocks - 1 - i);
    p->seg_of.assign(cfg->num_blocks, -1);
    if (!p->dry_run) p->append_of.assign(cfg->num_blocks, -1);
    *out = p;
    return APAR_OK;
}

int apar_pool_destroy(apar_pool* p) {
    if (!p) return APAR_OK;
    if (p->dry_run) {
        delete p;
        return APAR_OK;
    }
    DeviceGuard guard(p->device);
    int rc = APAR_OK;
    if (!hip_ok(hipDeviceSynchronize(), "hipDeviceSynchronize")) rc = APAR_ERR_HIP;
    release_workspace(p);
    if (p->copy_stream) (void)hipStreamDestroy(p->copy_stream);
    if (p->part.o) (void)hipFree(p->part.o);
    if (p->part.ml) (void)hipFree(p->part.ml);
    auto drop = [](hipEvent_t e) {
        if (e) (void)hipEventDestroy(e);
    };
    for (EventPair& e : p->decode_events) drop(e.a), drop(e.b), drop(e.c);
    for (EventPair& e : p->append_events) drop(e.a), drop(e.b), drop(e.c);
    for (hipEvent_t e : p->spare_events) drop(e);
    delete p;
    return rc;
}

int apar_thread_create(apar_pool* p, apar_thread* out) {
    if (!p || !out) return APAR_ERR_INVALID_ARG;
    if ((int64_t)p->threads.size() >= p->cfg.max_threads) return APAR_ERR_THREAD_CAPACITY;
    p->threads.emplace_back();
    p->threads.back().live = true;
    p->live_threads += 1;
    *out = (apar_thread)(p->threads.size() - 1);
    return APAR_OK;
}

int apar_fork(apar_pool* p, apar_thread parent, int n_children, apar_thread* children_out) {
    if (!p || !children_out) return APAR_ERR_INVALID_ARG;
    if (!live_thread(p, parent)) return APAR_ERR_INVALID_THREAD;
    if (n_children < 1) return APAR_ERR_INVALID_ARG;
    if ((int64_t)p->threads.size() + n_children > p->cfg.max_threads) return APAR_ERR_THREAD_CAPACITY;
    // (no exact-size reserve here: it would re-allocate the whole thread array on every fork)
    for (int c = 0; c < n_children; ++c) {
        p->threads.emplace_back();
        Thread& child = p->threads.back();
        const Thread& par = p->threads[parent];
        child.live = true;
        child.len = par.len;
        child.forked_from = parent;
        child.table = par.table;
        children_out[c] = (apar_thread)(p->threads.size() - 1);
    }
    for (int32_t b : p->threads[parent].table) p->ref[b] += n_children;
    p->live_threads += n_children;
    return APAR_OK;
}

int apar_append_kv(apar_pool* p, apar_thread thread, const void* k_dev, const void* v_dev, int n_tokens,
                   void* hip_stream) {
    if (!p || n_tokens < 0) return APAR_ERR_INVALID_ARG;
    Thread* t = live_thread(p, thread);
    if (!t) return APAR_ERR_INVALID_THREAD;
    if (n_tokens == 0) return APAR_OK;
    if (p->dry_run ? (k_dev || v_dev) : (!k_dev || !v_dev)) return APAR_ERR_INVALID_ARG;
    const int64_t B = kBlockTokens;
    int64_t need = (t->len + n_tokens + B - 1) / B - (t->len + B - 1) / B;
    if (t->len % B != 0 && p->ref[t->table.back()] > 1) need += 1;
    if (need > (int64_t)p->free_stack.size()) return APAR_ERR_OUT_OF_BLOCKS;
    std::vector<int32_t> codes(n_tokens), copies, seals;
    for (int i = 0; i < n_tokens; ++i) codes[i] = append_one(p, *t, copies, seals);
    if (p->check_writes && writes_are_private(p, codes, copies, seals) != APAR_OK) return APAR_ERR_INTERNAL;
    if (p->dry_run) return APAR_OK;
    DeviceGuard guard(p->device);
    return run_append(p, codes, copies, nullptr, k_dev, v_dev, (hipStream_t)hip_stream);
}

// One row per entry of `threads` (a thread may repeat), row i taken from row src_rows[i] of k_dev, v_dev
// (row i if src_rows is null).  All or nothing.
static int append_rows_of(apar_pool* p, const apar_thread* threads, int n, const std::vector<int32_t>* src_rows,
                          const void* k_dev, const void* v_dev, void* hip_stream) {
    if ((int64_t)p->free_stack.size() < n) {
        // Each row takes at most one block, so only a nearly full pool needs the
        // exact count: replay the policy on scratch copies of what it reads.
        struct Sim {
            int64_t len;
            bool private_tail;  // an earlier row of this call already made the tail this thread's own
        };
        std::unordered_map<int32_t, Sim> sim;         // by thread id
        std::unordered_map<int32_t, int32_t> dropped;  // references copy-on-write took off a block so far
        int64_t need = 0;
        for (int i = 0; i < n; ++i) {
            const Thread& t = p->threads[threads[i]];
            auto it = sim.find(threads[i]);
            if (it == sim.end()) it = sim.emplace(threads[i], Sim{t.len, false}).first;
            Sim& s = it->second;
            if (s.len % kBlockTokens == 0) {
                need += 1;
                s.private_tail = true;
            } else if (!s.private_tail) {
                const int32_t tail = t.table.back();
                int32_t& d = dropped[tail];
                if (p->ref[tail] - d > 1) {
                    need += 1;
                    d += 1;
                    s.private_tail = true;
                }
            }
            s.len += 1;
        }
        if (need > (int64_t)p->free_stack.size()) return APAR_ERR_OUT_OF_BLOCKS;
    }
    std::vector<int32_t>& codes = p->scratch_codes;
    std::vector<int32_t>& copies = p->scratch_copies;
    std::vector<int32_t>& seals = p->scratch_seals;
    codes.resize(n);
    copies.clear();
    seals.clear();
    for (int i = 0; i < n; ++i) codes[i] = append_one(p, p->threads[threads[i]], copies, seals);
    if (p->check_writes && writes_are_private(p, codes, copies, seals) != APAR_OK) return APAR_ERR_INTERNAL;
    if (p->dry_run) return APAR_OK;
    DeviceGuard guard(p->device);
    return run_append(p, codes, copies, src_rows, k_dev, v_dev, (hipStream_t)hip_stream);
}

int apar_append_kv_batch(apar_pool* p, const apar_thread* threads, int n, const void* k_dev, const void* v_dev,
                         void* hip_stream) {
    if (!p || n < 0) return APAR_ERR_INVALID_ARG;
    if (n == 0) return APAR_OK;
    if (!threads) return APAR_ERR_INVALID_ARG;
    if (p->dry_run ? (k_dev || v_dev) : (!k_dev || !v_dev)) return APAR_ERR_INVALID_ARG;
    for (int i = 0; i < n; ++i)
        if (!live_thread(p, threads[i])) return APAR_ERR_INVALID_THREAD;
    return append_rows_of(p, threads, n, nullptr, k_dev, v_dev, hip_stream);
}

int apar_append_kv_gather(apar_pool* p, const apar_thread* threads, const int32_t* src_rows, int n, const void* k_dev,
                          const void* v_dev, void* hip_stream) {
    if (!p || n < 0) return APAR_ERR_INVALID_ARG;
    if (n == 0) return APAR_OK;
    if (!threads || !src_rows) return APAR_ERR_INVALID_ARG;
    if (p->dry_run ? (k_dev || v_dev) : (!k_dev || !v_dev)) return APAR_ERR_INVALID_ARG;
    for (int i = 0; i < n; ++i) {
        if (!live_thread(p, threads[i])) return APAR_ERR_INVALID_THREAD;
        if (src_rows[i] < 0) return APAR_ERR_INVALID_ARG;
    }
    std::vector<int32_t>& src = p->scratch_commit_src;
    src.assign(src_rows, src_rows + n);
    return append_rows_of(p, threads, n, &src, k_dev, v_dev, hip_stream);
}

int apar_commit_candidates(apar_pool* p, const apar_thread* threads, int n, const void* cand_k_dev,
                           const void* cand_v_dev, int n_cand, const uint8_t* accept_masks, void* hip_stream) {
    if (!p || n < 0 || n_cand < 1 || n_cand > 8) return APAR_ERR_INVALID_ARG;
    if (n == 0) return APAR_OK;
    if (!threads || !accept_masks) return APAR_ERR_INVALID_ARG;
    if (p->dry_run ? (cand_k_dev || cand_v_dev) : (!cand_k_dev || !cand_v_dev)) return APAR_ERR_INVALID_ARG;
    if ((int64_t)n * n_cand > INT32_MAX) return APAR_ERR_INVALID_ARG;
    std::vector<apar_thread>& ids = p->scratch_commit_ids;
    std::vector<int32_t>& src = p->scratch_commit_src;
    ids.clear();
    src.clear();
    for (int i = 0; i < n; ++i) {
        if (!live_thread(p, threads[i])) return APAR_ERR_INVALID_THREAD;
        const uint32_t bits = accept_masks[i];
        if (bits >> n_cand) return APAR_ERR_INVALID_ARG;  // a candidate that does not exist
        for (int c = 0; c < n_cand; ++c)
            if ((bits >> c) & 1u) {
                ids.push_back(threads[i]);
                src.push_back(i * n_cand + c);
            }
    }
    if (ids.empty()) return APAR_OK;
    return append_rows_of(p, ids.data(), (int)ids.size(), &src, cand_k_dev, cand_v_dev, hip_stream);
}

int apar_decode_attention(apar_pool* p, const void* q_dev, const apar_thread* threads, int n, void* out_dev,
                          void* hip_stream) {
    return decode_common(p, q_dev, nullptr, nullptr, nullptr, 1, threads, n, out_dev, hip_stream, false);
}

int apar_decode_attention_spec(apar_pool* p, const void* q_dev, const void* cand_k_dev, const void* cand_v_dev,
                               const uint8_t* mask_dev, int n_cand, const apar_thread* threads, int n, void* out_dev,
                               void* hip_stream) {
    return decode_common(p, q_dev, cand_k_dev, cand_v_dev, mask_dev, n_cand, threads, n, out_dev, hip_stream, true);
}

int apar_decode_attention_fixed(apar_pool* p, const void* q_dev, const apar_thread* threads, int n, void* out_dev,
                                void* hip_stream) {
    return decode_common(p, q_dev, nullptr, nullptr, nullptr, 1, threads, n, out_dev, hip_stream, false, true);
}

int apar_prefill_attention(apar_pool* p, const void* q_dev, const apar_thread* threads, const int32_t* m, int n,
                           void* out_dev, void* hip_stream) {
    return prefill_common(p, q_dev, threads, m, n, out_dev, hip_stream);
}

int apar_free_thread(apar_pool* p, apar_thread thread) {
    if (!p) return APAR_ERR_INVALID_ARG;
    Thread* t = live_thread(p, thread);
    if (!t) return APAR_ERR_INVALID_THREAD;
    for (size_t i = t->table.size(); i-- > 0;) {
        const int32_t b = t->table[i];
        if (--p->ref[b] == 0) p->free_stack.push_back(b);
    }
    t->live = false;
    t->len = 0;
    std::vector<int32_t>().swap(t->table);
    p->live_threads -= 1;
    return APAR_OK;
}

int apar_thread_len(apar_pool* p, apar_thread thread, int64_t* len_out) {
    if (!p || !len_out) return APAR_ERR_INVALID_ARG;
    Thread* t = live_thread(p, thread);
    if (!t) return APAR_ERR_INVALID_THREAD;
    *len_out = t->len;
    return APAR_OK;
}

int apar_thread_block_table(apar_pool* p, apar_thread thread, int32_t* table_out, int cap, int* n_out) {
    if (!p || !n_out || cap < 0 || (cap > 0 && !table_out)) return APAR_ERR_INVALID_ARG;
    Thread* t = live_thread(p, thread);
    if (!t) return APAR_ERR_INVALID_THREAD;
    *n_out = (int)t->table.size();
    if ((size_t)cap < t->table.size()) return APAR_ERR_INVALID_ARG;
    if (!t->table.empty()) memcpy(table_out, t->table.data(), t->table.size() * sizeof(int32_t));
    return APAR_OK;
}

int apar_block_refcount(apar_pool* p, int32_t block, int32_t* refcount_out) {
    if (!p || !refcount_out || block < 0 || block >= p->cfg.num_blocks) return APAR_ERR_INVALID_ARG;
    *refcount_out = p->ref[block];
    return APAR_OK;
}

int apar_pool_stats(apar_pool* p, apar_stats* out) {
    if (!p || !out) return APAR_ERR_INVALID_ARG;
    out->total_blocks = p->cfg.num_blocks;
    out->free_blocks = (int64_t)p->free_stack.size();
    out->used_blocks = out->total_blocks - out->free_blocks;
    out->live_threads = p->live_threads;
    out->threads_issued = (int64_t)p->threads.size();
    out->cow_copies = p->cow_copies;
    out->block_bytes = p->shape.block_bytes;
    out->bytes_resident = out->used_blocks * p->shape.block_bytes;
    int64_t vanilla = 0;
    for (const Thread& t : p->threads)
        if (t.live) vanilla += (int64_t)t.table.size();
    out->bytes_vanilla = vanilla * p->shape.block_bytes;
    return APAR_OK;
}

int apar_last_plan_info(apar_pool* p, apar_plan_info* out) {
    if (!p || !out) return APAR_ERR_INVALID_ARG;
    *out = p->last_plan;
    return APAR_OK;
}

int apar_last_plan_export(apar_pool* p, int which, int32_t* out, int64_t cap, int64_t* n_out) {
    if (!p || !n_out || cap < 0 || (cap > 0 && !out)) return APAR_ERR_INVALID_ARG;
    const PlanHost& ph = p->plan;
    const int32_t* src = nullptr;
    int64_t n = 0;
    switch (which) {
        case APAR_PLAN_WORKGROUPS: src = (const int32_t*)ph.wgs.data(), n = (int64_t)ph.wgs.size() * 32; break;
        case APAR_PLAN_TILES: src = (const int32_t*)ph.tiles.data(), n = (int64_t)ph.tiles.size() * 2; break;
        case APAR_PLAN_DFS_THREADS: src = ph.dfs_threads.data(), n = (int64_t)ph.dfs_threads.size(); break;
        case APAR_PLAN_PATH_OFS: src = ph.path_ofs.data(), n = (int64_t)ph.path_ofs.size(); break;
        case APAR_PLAN_PATH_IDS: src = ph.path_ids.data(), n = (int64_t)ph.path_ids.size(); break;
        case APAR_PLAN_GEOMETRY: src = p->plan_geom, n = 3; break;
        case APAR_PLAN_CHANGED_WORKGROUP_WORDS: src = ph.dirty_wg_words.data(), n = (int64_t)ph.dirty_wg_words.size(); break;
        case APAR_PLAN_CHANGED_TILE_WORDS: src = ph.dirty_tile_words.data(), n = (int64_t)ph.dirty_tile_words.size(); break;
        default: return APAR_ERR_INVALID_ARG;
    }
    *n_out = n;
    if (cap < n) return APAR_ERR_INVALID_ARG;
    if (n > 0) memcpy(out, src, (size_t)n * sizeof(int32_t));
    return APAR_OK;
}

int apar_read_kv_rows(apar_pool* p, apar_thread thread, int64_t first, int n, void* k_out_dev, void* v_out_dev,
                      void* hip_stream) {
    if (!p || n < 0 || first < 0) return APAR_ERR_INVALID_ARG;
    Thread* t = live_thread(p, thread);
    if (!t) return APAR_ERR_INVALID_THREAD;
    if (first + n > t->len || p->dry_run) return APAR_ERR_INVALID_ARG;
    if (n == 0) return APAR_OK;
    if (!k_out_dev || !v_out_dev) return APAR_ERR_INVALID_ARG;
    DeviceGuard guard(p->device);
    hipStream_t st = (hipStream_t)hip_stream;
    StageSlot* s = nullptr;
    int rc = acquire_stage(p, (size_t)n * sizeof(int32_t), &s);
    if (rc != APAR_OK) return rc;
    int32_t* codes = (int32_t*)s->host;
    for (int i = 0; i < n; ++i) {
        const int64_t pos = first + i;
        const bool sealed = p->shape.dtype == APAR_BF16 && (pos / kBlockTokens + 1) * kBlockTokens <= t->len;
        codes[i] = slot_code(*t, pos) | (sealed ? kCodeSealed : 0);
    }
    if ((rc = upload(p, s, (size_t)n * sizeof(int32_t), st)) != APAR_OK) return rc;
    HIP_TRY(launch_read_rows(p->shape, p->kv, (const int32_t*)s->dev, n, k_out_dev, v_out_dev, st));
    HIP_TRY(hipEventRecord(s->ev, st));
    s->pending = true;
    return APAR_OK;
}

int apar_profile_enable(apar_pool* p, int on) {
    if (!p) return APAR_ERR_INVALID_ARG;
    p->profiling = on != 0;
    return APAR_OK;
}

int apar_profile_read(apar_pool* p, apar_profile* out) {
    if (!p || !out) return APAR_ERR_INVALID_ARG;
    memset(out, 0, sizeof(*out));
    p->last_attention_ms.clear();
    if (p->dry_run) return APAR_OK;
    DeviceGuard guard(p->device);
    for (EventPair& e : p->decode_events) {
        float ms = 0.0f;
        HIP_TRY(hipEventSynchronize(e.c));
        HIP_TRY(hipEventElapsedTime(&ms, e.a, e.b));
        out->attention_kernel_ms += ms;
        p->last_attention_ms.push_back(ms);
        HIP_TRY(hipEventElapsedTime(&ms, e.b, e.c));
        out->merge_kernel_ms += ms;
        p->spare_events.push_back(e.a);
        p->spare_events.push_back(e.b);
        p->spare_events.push_back(e.c);
    }
    for (EventPair& e : p->append_events) {
        float ms = 0.0f;
        HIP_TRY(hipEventSynchronize(e.b));
        HIP_TRY(hipEventElapsedTime(&ms, e.a, e.b));
        out->append_kernels_ms += ms;
        p->spare_events.push_back(e.a);
        p->spare_events.push_back(e.b);
    }
    out->n_decode_calls = p->n_decode_calls;
    out->n_append_calls = p->n_append_calls;
    out->plan_host_ms = p->plan_host_ms;
    out->host_wait_ms = p->host_wait_ms;
    p->decode_events.clear();
    p->append_events.clear();
    p->n_decode_calls = p->n_append_calls = 0;
    p->plan_host_ms = p->host_wait_ms = 0.0;
    return APAR_OK;
}

int apar_profile_attention_calls(apar_pool* p, float* ms_out, int64_t cap, int64_t* n_out) {
    if (!p || !n_out || cap < 0 || (cap > 0 && !ms_out)) return APAR_ERR_INVALID_ARG;
    const int64_t n = (int64_t)p->last_attention_ms.size();
    *n_out = n;
    if (cap < n) return APAR_ERR_INVALID_ARG;
    if (n > 0) memcpy(ms_out, p->last_attention_ms.data(), (size_t)n * sizeof(float));
    return APAR_OK;
}

int apar_plan_record_version(void) { return APAR_PLAN_RECORD_VERSION; }

int apar_set_plan_reuse(apar_pool* p, int on) {
    if (!p) return APAR_ERR_INVALID_ARG;
    p->plan_reuse = on != 0;
    return APAR_OK;
}

int apar_plan_counts(apar_pool* p, int64_t* n_built, int64_t* n_carried) {
    if (!p || !n_built || !n_carried) return APAR_ERR_INVALID_ARG;
    *n_built = p->n_plans_built;
    *n_carried = p->n_plans_carried;
    return APAR_OK;
}

int apar_set_write_checks(apar_pool* p, int on) {
    if (!p) return APAR_ERR_INVALID_ARG;
    p->check_writes = on != 0;
    return APAR_OK;
}

int apar_set_inline_shared(apar_pool* p, int on) {
    if (!p) return APAR_ERR_INVALID_ARG;
    p->inline_shared = on != 0;
    p->planning_set = true;
    return APAR_OK;
}

int apar_set_matrix_units(apar_pool* p, int min_rows, int min_blocks) {
    if (!p || min_rows < 0 || min_blocks < 0) return APAR_ERR_INVALID_ARG;
    p->matrix_min_rows = min_rows;
    p->matrix_min_blocks = min_blocks;
    p->planning_set = p->planning_set || p->has_matrix_units();  // (other pools ignore the knob)
    return APAR_OK;
}

int apar_set_prefill_kernel(apar_pool* p, int which) {
    if (!p || which < APAR_PREFILL_AUTO || which > APAR_PREFILL_MATRIX) return APAR_ERR_INVALID_ARG;
    p->prefill_kernel = which;
    return APAR_OK;
}

int apar_last_prefill_kernel(apar_pool* p) { return p ? p->last_prefill_kernel : 0; }

int apar_set_chunk_blocks(apar_pool* p, int blocks_per_unit) {
    if (!p || blocks_per_unit < 1 || blocks_per_unit > 65536) return APAR_ERR_INVALID_ARG;
    p->max_unit_tiles = blocks_per_unit;
    p->planning_set = true;
    return APAR_OK;
}

const char* apar_status_string(int status) {
    switch (status) {
        case APAR_OK: return "ok";
        case APAR_ERR_INVALID_ARG: return "invalid argument";
        case APAR_ERR_INVALID_THREAD: return "invalid thread";
        case APAR_ERR_OUT_OF_BLOCKS: return "out of blocks";
        case APAR_ERR_THREAD_CAPACITY: return "thread capacity exceeded";
        case APAR_ERR_HIP: return "HIP runtime error";
        case APAR_ERR_UNSUPPORTED: return "unsupported shape";
        case APAR_ERR_WORKSPACE_LIMIT: return "call exceeds the fixed workspace";
        case APAR_ERR_INTERNAL: return "internal invariant violated";
        default: return "unknown status";
    }
}

const char* apar_last_hip_error(void) { return g_last_hip_error.c_str(); }

}  // extern "C"
