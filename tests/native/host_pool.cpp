// The host side of a pool that launches, against a HIP runtime that runs on the host: allocations are counted and can be
// refused, copies happen at once, kernels only look at what they were handed.  Built and run by
// tests/test_pool_resources.py, which names the check to run.
#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <string>
#include <vector>

#include "apar_internal.hpp"

#define CHECK(c)                                                              \
    do {                                                                      \
        if (!(c)) {                                                           \
            std::fprintf(stderr, "check failed: %s (line %d)\n", #c, __LINE__); \
            std::exit(1);                                                     \
        }                                                                     \
    } while (0)

// ---- the runtime ------------------------------------------------------------------------------------
static std::map<char*, size_t> g_dev, g_host;      // live allocations
static int g_allocs = 0, g_refuse = -1;            // allocations so far; the one to refuse (-1: none)
static bool g_refuse_rest = false;                 // ... and all after it
static int g_waits = 0, g_objects = 0;             // calls that wait for the device; live events and streams
static bool g_capturing = false;
static hipError_t g_last = hipSuccess;

static hipError_t failed(hipError_t e) { return g_last = e; }
static hipError_t allocate(std::map<char*, size_t>& live, void** out, size_t size) {
    const int n = g_allocs++;
    if (n == g_refuse || (g_refuse_rest && g_refuse >= 0 && n > g_refuse)) return failed(hipErrorOutOfMemory);
    char* p = (char*)std::aligned_alloc(256, (size + 255) / 256 * 256);
    std::memset(p, 0xa5, size);
    live[p] = size;
    *out = p;
    return hipSuccess;
}
static hipError_t release(std::map<char*, size_t>& live, void* p) {
    if (!p) return hipSuccess;
    g_waits += 1;
    CHECK(live.erase((char*)p) == 1);
    std::free(p);
    return hipSuccess;
}
static bool on_device(const void* p, size_t bytes) {
    auto it = g_dev.upper_bound((char*)p);
    return it != g_dev.begin() && (--it, (char*)p + bytes <= it->first + it->second);
}
extern "C" {
hipError_t hipMalloc(void** p, size_t size) { return allocate(g_dev, p, size); }
hipError_t hipFree(void* p) { return release(g_dev, p); }
hipError_t hipHostMalloc(void** p, size_t size, unsigned int) { return allocate(g_host, p, size); }
hipError_t hipHostFree(void* p) { return release(g_host, p); }
hipError_t hipMemcpy(void* d, const void* s, size_t n, hipMemcpyKind) { g_waits += 1; std::memcpy(d, s, n); return hipSuccess; }
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind, hipStream_t) { std::memcpy(d, s, n); return hipSuccess; }
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus* s) { *s = g_capturing ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone; return hipSuccess; }
hipError_t hipDeviceSynchronize() { g_waits += 1; return hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { g_objects += 1; *e = (hipEvent_t)std::malloc(1); return hipSuccess; }
hipError_t hipEventCreate(hipEvent_t* e) { return hipEventCreateWithFlags(e, 0); }
hipError_t hipEventDestroy(hipEvent_t e) { g_objects -= 1; std::free((void*)e); return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t e, hipStream_t) { CHECK(e != nullptr); return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }  // (a slot's last kernels: done by then)
hipError_t hipEventElapsedTime(float* ms, hipEvent_t, hipEvent_t) { *ms = 0.0f; return hipSuccess; }
hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) { g_objects += 1; *s = (hipStream_t)std::malloc(1); return hipSuccess; }
hipError_t hipStreamDestroy(hipStream_t s) { g_objects -= 1; std::free((void*)s); return hipSuccess; }
hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned) { return hipSuccess; }
hipError_t hipGetDevice(int* d) { *d = 0; return hipSuccess; }
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipGetLastError() { const hipError_t e = g_last; g_last = hipSuccess; return e; }
const char* hipGetErrorString(hipError_t) { return "refused"; }
hipError_t hipPointerGetAttributes(hipPointerAttribute_t* a, const void*) { *a = hipPointerAttribute_t{}; return hipSuccess; }
}

// ---- the kernels ------------------------------------------------------------------------------------
static apar::PlanDev g_plan;  // of the last decode or row-tile prefill call
static std::vector<apar::SplitBlock> g_blocks;
static apar::PartialBuf g_part;
static int g_clears = 0;  // launches that cleared counters
static char* g_fixed = nullptr;
namespace apar {
hipError_t fixed_workspace_of_device(int, char** out) {
    if (!g_fixed) g_fixed = (char*)std::aligned_alloc(256, (size_t)APAR_FIXED_PLAN_BYTES + APAR_FIXED_PARTIAL_BYTES);
    *out = g_fixed;
    return hipSuccess;
}
hipError_t launch_append_blocks(const Shape&, void*, const void*, const void*, const int32_t*, bool, int, int, int, hipStream_t) { return hipGetLastError(); }
hipError_t launch_block_copies(const Shape&, void*, const int32_t*, int, hipStream_t) { return hipGetLastError(); }
hipError_t launch_read_rows(const Shape&, const void*, const int32_t* codes, int n, void*, void*, hipStream_t) {
    CHECK(on_device(codes, (size_t)n * 4));
    return hipGetLastError();
}
hipError_t launch_scatter_words(int32_t*, const int32_t*, int, hipStream_t) { return hipGetLastError(); }
hipError_t launch_clear_words(int32_t* words, int n, hipStream_t) {
    CHECK(on_device(words, (size_t)n * 4));
    std::memset(words, 0, (size_t)n * 4);
    g_clears += 1;
    return hipGetLastError();
}
// Every cut unit's states and counters lie in memory of their own, and no unit is cut without room for them.
hipError_t launch_attention_partial(const Shape& s, const void*, const void*, const PlanDev& plan, int, PartialBuf part, const void*, const void*,
                                    const uint8_t*, void*, hipStream_t) {
    g_plan = plan;
    g_part = part;
    g_blocks.clear();
    if (plan.split.blocks) {
        const char* base = plan.inline_words ? (const char*)plan.inline_words : nullptr;
        const SplitBlock* b = (const SplitBlock*)(base + (size_t)plan.split.blocks);
        const WgDesc* wgs = (const WgDesc*)(base + (size_t)plan.wgs);
        g_blocks.assign(b, b + plan.split.n_blocks_class[0] + plan.split.n_blocks_class[1] + plan.split.n_blocks_class[2]);
        int state = 0, cut = 0;
        for (const SplitBlock& x : g_blocks) {  // a unit's slices in a row, its states and counters behind those of the unit before
            const int at = (int)(&x - g_blocks.data()), n_of = x.slice >> 16, s_of = x.slice & 0xffff;
            CHECK(s_of < n_of && x.state == state && x.cut == cut);
            CHECK(at == 0 ? x.wg == 0 && s_of == 0 : s_of == 0 ? x.wg == g_blocks[at - 1].wg + 1 : x.wg == g_blocks[at - 1].wg && s_of == (g_blocks[at - 1].slice & 0xffff) + 1);
            if (n_of > 1 && s_of == n_of - 1) state += n_of * (wgs[x.wg].w[0].flags & kWaveSplit ? 1 : 4) * (wgs[x.wg].row_tiles & 255), cut += 1;
        }
        CHECK(g_blocks.empty() || ((g_blocks.back().slice & 0xffff) == (g_blocks.back().slice >> 16) - 1 && g_blocks.back().wg == plan.n_wg - 1));
        for (const SplitBlock& x : g_blocks) {
            const int n = x.slice >> 16, tiles = (wgs[x.wg].w[0].flags & kWaveSplit ? 1 : 4) * (wgs[x.wg].row_tiles & 255);
            if (n == 1) continue;
            const size_t tile = (size_t)(s.d / 4 + 2) * 64 * 4;
            CHECK(on_device((char*)plan.split.state + (size_t)x.state * s.n_kv * tile, (size_t)n * tiles * s.n_kv * tile));
            const int32_t* counters = plan.split.arrived + (size_t)x.cut * s.n_kv * 4;
            CHECK(on_device(counters, (size_t)s.n_kv * 16));
            for (int i = 0; i < s.n_kv * 4; ++i) CHECK(counters[i] == 0);
        }
    }
    return hipGetLastError();
}
hipError_t launch_prefill_bf16(const Shape&, const void*, const void*, const PrefillWg*, const int32_t*, int, void*, hipStream_t) { return hipGetLastError(); }
hipError_t launch_merge(const Shape&, const PlanDev&, PartialBuf, const void*, const void*, const void*, const uint8_t*, int, void*, hipStream_t) {
    return hipGetLastError();
}
}  // namespace apar

// ---- checks -----------------------------------------------------------------------------------------
static char g_kv[256] __attribute__((aligned(256)));  // (no kernel runs: the pool's memory is never touched)
static void* const kRows = g_kv;

static int create(int n_q, int n_kv, int dtype, int64_t blocks, apar_pool** p) {
    apar_pool_config c{};
    c.n_q_heads = n_q, c.n_kv_heads = n_kv, c.head_dim = 128, c.block_size = 16, c.dtype = dtype, c.max_threads = 1 << 20, c.num_blocks = blocks;
    const int waits = g_waits, rc = apar_pool_create(&c, g_kv, (size_t)1 << 60, p);
    CHECK(rc != APAR_OK || g_waits == waits);
    return rc;
}
static apar_thread thread_of(apar_pool* p, int n) {
    apar_thread t;
    CHECK(apar_thread_create(p, &t) == APAR_OK && apar_append_kv(p, t, kRows, kRows, n, nullptr) == APAR_OK);
    return t;
}

// Once a pool is there, its first calls neither allocate nor wait, whichever staging slot they come to.
static void staging() {
    apar_pool* p;
    CHECK(create(8, 8, APAR_BF16, 4000, &p) == APAR_OK);
    std::vector<apar_thread> ids;
    for (int i = 0; i < 120; ++i) ids.push_back(thread_of(p, 100 + i));
    const int allocs = g_allocs, waits = g_waits;
    for (int step = 0; step < 9; ++step) {
        CHECK(apar_decode_attention(p, kRows, ids.data(), (int)ids.size(), kRows, nullptr) == APAR_OK);
        CHECK(g_plan.inline_words == nullptr);  // (staged)
        CHECK(apar_read_kv_rows(p, ids[0], 0, 100, kRows, kRows, nullptr) == APAR_OK);
        CHECK(apar_append_kv_batch(p, ids.data(), (int)ids.size(), kRows, kRows, nullptr) == APAR_OK);
    }
    CHECK(g_allocs == allocs && g_waits == waits);
    // a larger request takes memory of its own, and still does not wait the first time
    const apar_thread big = thread_of(p, 40000);
    CHECK(apar_read_kv_rows(p, big, 0, 40000, kRows, kRows, nullptr) == APAR_OK);
    std::vector<int32_t> m(1, 40000);
    CHECK(g_waits == waits);
    CHECK(apar_pool_destroy(p) == APAR_OK);
    CHECK(g_dev.empty() && g_host.empty() && g_objects == 0);
}

// What a pool works in besides its blocks is only needed by some calls: whichever allocation is refused, alone or with
// all after it, creation succeeds as long as the buffer of the entry point that may not allocate is there.
static void creation() {
    for (int rest = 0; rest < 2; ++rest)
        for (int k = 0; k < 4; ++k) {
            apar_pool* p = nullptr;
            g_allocs = 0, g_refuse = k, g_refuse_rest = rest != 0;
            const int rc = create(8, 8, APAR_BF16, 4000, &p);
            const bool room = k > 0;  // (the device allocation comes first)
            g_refuse = -1;
            CHECK(rc == (rest && k <= 1 ? APAR_ERR_HIP : APAR_OK) && (rc == APAR_OK) == (p != nullptr));
            if (p) {
                const apar_thread t = thread_of(p, 1600);
                CHECK(apar_decode_attention(p, kRows, &t, 1, kRows, nullptr) == APAR_OK);  // (a long walk: cut where there is room)
                int slices = 0;
                for (const apar::SplitBlock& b : g_blocks) slices = std::max(slices, b.slice >> 16);
                CHECK((slices > 1) == room);
                CHECK(apar_read_kv_rows(p, t, 0, 1600, kRows, kRows, nullptr) == APAR_OK);
            }
            CHECK(apar_pool_destroy(p) == APAR_OK && g_dev.empty() && g_host.empty() && g_objects == 0);
        }
}

// The entry point that may not allocate cuts as the other does, its states in the pool's own memory: the workspace that is
// part of the device image holds tables and partial results, nothing after them.
static void fixed() {
    apar_pool* p;
    CHECK(create(8, 8, APAR_BF16, 4000, &p) == APAR_OK);
    const apar_thread t = thread_of(p, 1600);
    for (int k = 0; k < 2; ++k) {
        CHECK(apar_decode_attention(p, kRows, &t, 1, kRows, nullptr) == APAR_OK);
        const std::vector<apar::SplitBlock> as = g_blocks;
        const int allocs = g_allocs;
        CHECK(apar_decode_attention_fixed(p, kRows, &t, 1, kRows, nullptr) == APAR_OK);  // (where the states lie: at the launch)
        CHECK(g_allocs == allocs && as.size() > 1 && as.size() == g_blocks.size());
        for (size_t i = 0; i < as.size(); ++i) CHECK(std::memcmp(&as[i], &g_blocks[i], sizeof as[i]) == 0);
    }
    CHECK(apar_pool_destroy(p) == APAR_OK);
    // the counters are cleared once, but not by a call that is only recorded: its clear belongs to the graph
    CHECK(create(8, 8, APAR_BF16, 4000, &p) == APAR_OK);
    const apar_thread u0 = thread_of(p, 1600);
    g_clears = 0, g_capturing = true;
    for (int k = 0; k < 2; ++k) CHECK(apar_decode_attention_fixed(p, kRows, &u0, 1, kRows, nullptr) == APAR_OK && g_clears == k + 1);
    g_capturing = false;
    for (int k = 0; k < 2; ++k) CHECK(apar_decode_attention_fixed(p, kRows, &u0, 1, kRows, nullptr) == APAR_OK && g_clears == 3);
    CHECK(apar_decode_attention(p, kRows, &u0, 1, kRows, nullptr) == APAR_OK && g_clears == 3);
    CHECK(apar_pool_destroy(p) == APAR_OK);
    // one long thread beside so many short ones that the tables come to the limit: cut, then whole, then refused
    int seen[3] = {0, 0, 0};
    for (int n = 22000; n < 32000; n += 2000) {
        CHECK(create(1, 1, APAR_BF16, 40000, &p) == APAR_OK);
        std::vector<apar_thread> ids(1, thread_of(p, 16000));
        apar_thread u;
        for (int i = 0; i < n; ++i) {
            CHECK(apar_thread_create(p, &u) == APAR_OK);
            ids.push_back(u);
        }
        CHECK(apar_append_kv_batch(p, ids.data() + 1, n, kRows, kRows, nullptr) == APAR_OK);
        const int rc = apar_decode_attention_fixed(p, kRows, ids.data(), n + 1, kRows, nullptr);
        CHECK(rc == APAR_OK || rc == APAR_ERR_WORKSPACE_LIMIT);
        const int at = rc != APAR_OK ? 2 : g_blocks.empty() ? 1 : 0;
        for (int later = at + 1; later < 3; ++later) CHECK(seen[later] == 0);
        seen[at] += 1;
        if (rc == APAR_OK) {  // (the other entry point cuts)
            CHECK(apar_decode_attention(p, kRows, ids.data(), n + 1, kRows, nullptr) == APAR_OK && !g_blocks.empty());
        }
        CHECK(apar_pool_destroy(p) == APAR_OK);
    }
    CHECK(seen[0] && seen[1] && seen[2]);
}

// Units are cut as far as there is room for their states, down to not at all, and always completely (at the launch).
static int longest_cut(int n_q, int n_kv, int dtype, int64_t blocks, int root, int kids, int kid_len) {
    apar_pool* p;
    CHECK(create(n_q, n_kv, dtype, blocks, &p) == APAR_OK);
    const apar_thread t = thread_of(p, root);
    std::vector<apar_thread> ids(kids + 1);
    CHECK(apar_fork(p, t, kids, ids.data()) == APAR_OK);
    ids[kids] = t;
    for (int i = 0; i < kids; ++i) CHECK(apar_append_kv(p, ids[i], kRows, kRows, kid_len > 1 ? kid_len + i % 30 : 1, nullptr) == APAR_OK);
    CHECK(apar_decode_attention(p, kRows, ids.data(), kids + 1, kRows, nullptr) == APAR_OK);
    int slices = 1;
    for (const apar::SplitBlock& b : g_blocks) slices = std::max(slices, b.slice >> 16);
    const int rc = apar_decode_attention_fixed(p, kRows, ids.data(), kids + 1, kRows, nullptr);
    CHECK(rc == APAR_OK || rc == APAR_ERR_WORKSPACE_LIMIT);
    CHECK(apar_pool_destroy(p) == APAR_OK);
    return slices;
}
static void slices() {
    for (int dtype : {APAR_F32, APAR_BF16})
        for (int n_kv : {1, 4, 32})
            for (int kids : {1, 5, 40, 150})
                for (int root : {40, 640, 6000}) longest_cut(n_kv * 4, n_kv, dtype, 200000, root, kids, 17);
    // seventy leaves below 640 rows, 16 kv heads: room for all, for fewer slices than that, for none
    const int all = longest_cut(16, 16, APAR_BF16, 100000, 640, 70, 16), some = longest_cut(16, 16, APAR_BF16, 290, 640, 70, 16);
    CHECK(all > some && some > 1 && longest_cut(16, 16, APAR_BF16, 114, 640, 70, 1) == 1);
}

// Partial results are streamed where the call's are more than the memory-side cache holds.
static void partials() {
    for (int n : {200, 3200}) {
        apar_pool* p;
        CHECK(create(32, 8, APAR_BF16, 100000, &p) == APAR_OK);
        CHECK(apar_set_chunk_blocks(p, 2) == APAR_OK);
        std::vector<apar_thread> ids;
        for (int i = 0; i < n; ++i) ids.push_back(thread_of(p, 200));
        CHECK(apar_decode_attention(p, kRows, ids.data(), n, kRows, nullptr) == APAR_OK);
        apar_plan_info info;
        CHECK(apar_last_plan_info(p, &info) == APAR_OK && info.n_partial_rows > n);
        CHECK((g_part.stream != 0) == (info.n_partial_rows * 32 * 520 > (int64_t)256 << 20) && (g_part.stream != 0) == (n == 3200));
        CHECK(apar_pool_destroy(p) == APAR_OK);
    }
}

// Which kernel a prefill call goes to by itself, on either side of the rule's lines (us on the row tiles / the matrix kernel, where
// six threads share a prefix).
static void prefill() {
    struct Call { int dtype, n_q, n_kv, threads, len, m, long_m, kernel; };  // long_m: one prompt of that many tokens besides
    const int T = APAR_PREFILL_ROW_TILES, M = APAR_PREFILL_MATRIX;
    const Call calls[] = {
        {APAR_BF16_FP8KV, 32, 32, 362, 380, 48, 0, T},  {APAR_BF16_FP8KV, 32, 32, 362, 380, 90, 0, M},  // 301 / 325, 503 / 365
        {APAR_BF16_FP8KV, 32, 4, 891, 380, 6, 0, T},    {APAR_BF16_FP8KV, 32, 4, 891, 380, 10, 0, M},   // 124 / 110, 169 / 124
        {APAR_BF16_FP8KV, 32, 8, 362, 1100, 16, 0, T},  {APAR_BF16_FP8KV, 32, 8, 362, 1100, 20, 0, M},  // 183 / 197, 290 / 215
        {APAR_BF16, 32, 8, 362, 300, 16, 0, T},         {APAR_BF16, 32, 8, 362, 300, 24, 0, M},         // 76 / 79, 115 / 84
        {APAR_BF16, 32, 16, 179, 700, 24, 0, T},        {APAR_BF16, 32, 16, 179, 700, 40, 0, M},        // 121 / 123, 197 / 142
        {APAR_BF16, 32, 32, 179, 380, 48, 0, T},        {APAR_BF16, 32, 32, 891, 700, 48, 0, M},        // 151 / 160, 1224 / 1172
        {APAR_BF16, 32, 32, 362, 300, 1, 0, T},         {APAR_BF16, 32, 32, 362, 1100, 1, 0, M},        // 166 / 215, 499 / 523
        {APAR_BF16, 32, 32, 360, 901, 1, 2000, T},      {APAR_BF16, 32, 4, 360, 301, 1, 2000, M},       // 556 / 477, 89 / 71
        {APAR_BF16_FP8KV, 32, 4, 360, 301, 1, 2000, M}, {APAR_BF16, 32, 8, 360, 901, 1, 2000, T},       // 91 / 75, 179 / 154
    };
    for (const Call& c : calls) {
        apar_pool* p;
        CHECK(create(c.n_q, c.n_kv, c.dtype, 70000, &p) == APAR_OK);
        std::vector<apar_thread> ids;
        for (int i = 0; i < c.threads; ++i) ids.push_back(thread_of(p, c.len));
        std::vector<int32_t> m(ids.size(), c.m);
        if (c.long_m) ids.push_back(thread_of(p, c.long_m)), m.push_back(c.long_m);
        CHECK(apar_prefill_attention(p, kRows, ids.data(), m.data(), (int)ids.size(), kRows, nullptr) == APAR_OK);
        if (apar_last_prefill_kernel(p) != c.kernel) std::fprintf(stderr, "call %d\n", (int)(&c - calls));
        CHECK(apar_last_prefill_kernel(p) == c.kernel);
        CHECK(apar_pool_destroy(p) == APAR_OK);
    }
}

int main(int argc, char** argv) {
    const std::map<std::string, void (*)()> checks = {{"staging", staging}, {"creation", creation}, {"fixed", fixed}, {"prefill", prefill}, {"slices", slices}, {"partials", partials}};
    CHECK(argc == 2 && checks.count(argv[1]));
    checks.at(argv[1])();
    std::printf("ok: %s\n", argv[1]);
    return 0;
}
