// The library's host code against a device that is not there: the HIP calls and the kernel launchers are replaced by functions
// that count, so that what a call asks the runtime for can be checked where no GPU is.  Built and run by
// tests/test_host_fake_device.py, a check of those in main at a time; exits non-zero on a mismatch.
#include <hip/hip_runtime_api.h>

#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <vector>

#include "../paper_2605_13784_amd/csrc/sk_pool.cpp"

#define CHECK(c) do { if (!(c)) { std::fprintf(stderr, "check failed at line %d: %s\n", __LINE__, #c); std::exit(1); } } while (0)

static int n_events, recorded[16], waited[16], copies, launch_error;
static unsigned host_flags;
static const void* list_at;
static std::vector<sk_work> work;            // of the last batched call's attention launches, and their other arguments
static std::vector<sk_launch> launches;
static std::vector<sk_comb> merges;

extern "C" {
hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t, int) { *v = 256; return hipSuccess; }
hipError_t hipDeviceSynchronize() { return hipSuccess; }
hipError_t hipEventCreate(hipEvent_t* e) { *e = (hipEvent_t)(intptr_t)++n_events; return hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { return hipEventCreate(e); }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float* t, hipEvent_t, hipEvent_t) { *t = 0.f; return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t e, hipStream_t) { ++recorded[(intptr_t)e]; return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t e) { ++waited[(intptr_t)e]; return hipSuccess; }
hipError_t hipGetDevice(int* d) { *d = 0; return hipSuccess; }
hipError_t hipHostFree(void* p) { std::free(p); return hipSuccess; }
hipError_t hipHostMalloc(void** p, size_t n, unsigned flags) { host_flags = flags; *p = std::malloc(n); return *p ? hipSuccess : hipErrorOutOfMemory; }
hipError_t hipMemcpy(void* d, const void* s, size_t n, hipMemcpyKind) { std::memcpy(d, s, n); return hipSuccess; }
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind, hipStream_t) { std::memcpy(d, s, n); ++copies; return hipSuccess; }
hipError_t hipMemset(void* d, int x, size_t n) { std::memset(d, x, n); return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
}
int sk_launch_scatter(const sk_geom&, const void*, const void*, const sk_scatter* items, int32_t n, int32_t*, unsigned char*, unsigned char* eph, void*)
{
    list_at = items;
    for (int32_t i = 0; i < n; ++i)          // what the kernel does with such an item
        if (items[i].to_eph == SK_COPY_LIST) std::memcpy(eph + items[i].dst_off, (const char*)items + 16 * (size_t)items[i].src_tok0, 16 * (size_t)items[i].count);
    const int e = launch_error;
    launch_error = 0;
    return e;
}
int sk_launch_scatter_args(const sk_geom&, const void*, const void*, const sk_scatter_list&, int32_t, int32_t*, unsigned char*, unsigned char*, void*) { return 0; }
int sk_launch_attention(const sk_launch& L, int, int32_t n, void*, void*, void*)
{
    launches.push_back(L);
    if (L.mode == SK_MODE_LIST) work.insert(work.end(), L.work, L.work + n);
    return 0;
}
int sk_launch_attention_small(const sk_launch& L, const sk_commit&, int32_t n, void*, void*, void*) { return sk_launch_attention(L, 0, n, nullptr, nullptr, nullptr); }
int sk_launch_combine(const sk_launch& L, int32_t n, int32_t, int64_t, void*, void*, void*)
{
    if (L.mode == SK_MODE_LIST) merges.insert(merges.end(), L.comb, L.comb + n);
    return 0;
}
int sk_launch_gather(const sk_geom&, int32_t, int64_t, int64_t, void*, void*, void*) { return 0; }
int sk_launch_copy_block(const sk_geom&, unsigned char*, int32_t, int32_t, void*) { return 0; }

static sk_pool* make_pool(sk_pool_desc& d, int dtype = SK_BF16)
{
    d.dtype = dtype; d.block_tokens = 16;
    d.kv_bytes = sk_pool_kv_bytes(&d); d.workspace_bytes = sk_pool_workspace_bytes(&d);
    d.kv_mem = std::aligned_alloc(256, (d.kv_bytes + 255) / 256 * 256);
    d.workspace = std::aligned_alloc(256, (d.workspace_bytes + 255) / 256 * 256);
    sk_pool* p = nullptr;
    CHECK(sk_pool_create(&d, &p) == SK_OK);
    return p;
}
static void drop_pool(sk_pool* p, sk_pool_desc& d) { CHECK(sk_pool_destroy(p) == SK_OK); std::free(d.kv_mem); std::free(d.workspace); }

static void check_ring()
{
    sk_pool_desc d = {};
    d.dtype = SK_BF16; d.n_q_heads = d.n_kv_heads = 1; d.head_dim = 64; d.block_tokens = 16; d.max_sessions = 1;
    d.n_blocks = 1 << 14; d.max_batch_tokens = 1 << 18;
    d.kv_bytes = sk_pool_kv_bytes(&d); d.workspace_bytes = sk_pool_workspace_bytes(&d);
    d.kv_mem = std::aligned_alloc(256, (d.kv_bytes + 255) / 256 * 256);
    d.workspace = std::aligned_alloc(256, (d.workspace_bytes + 255) / 256 * 256);
    sk_pool* p = nullptr;
    int32_t id = -1;
    CHECK(sk_pool_create(&d, &p) == SK_OK && sk_session_create(p, &id) == SK_OK);
    CHECK((host_flags & hipHostMallocCoherent) && (host_flags & hipHostMallocMapped));       // kernels read lists there
    const int slots = n_events;                     // one event per slot of the pinned ring, numbered from 1
    CHECK(slots >= 2 && slots < 16);
    static __attribute__((aligned(16))) char kv[16];
    auto append = [&](int32_t L) {
        const int rc = sk_session_append(p, id, nullptr, kv, kv, L, nullptr, SK_F32, nullptr, nullptr);
        if (rc == SK_OK) CHECK(sk_session_truncate(p, id, 0) == SK_OK);
        return rc;
    };
    // A launch reports the error that an earlier call of the thread left behind, and is on the stream all the same: the slot its
    // kernel reads stays busy, so the append that comes round to it waits.
    launch_error = (int)hipErrorInvalidValue;
    CHECK(append(1300) == SK_E_HIP && recorded[1] == 1);
    for (int i = 1; i < slots; ++i) CHECK(append(1300) == SK_OK && recorded[i + 1] == 1);
    CHECK(waited[1] == 0);
    CHECK(append(1300) == SK_OK && waited[1] == 1);
    // Up to 8,192 groups of 16 tokens the list is read where it lies, a longer one from the workspace, behind a copy.
    for (int32_t groups : {81, 8192, 8193, 9000}) {
        const int before = copies;
        CHECK(append(16 * groups) == SK_OK && copies - before == (groups > 8192 ? 1 : 0));
        const char* w = (const char*)d.workspace;
        CHECK(((const char*)list_at >= w && (const char*)list_at < w + d.workspace_bytes) == (groups > 8192));
        CHECK(((const sk_scatter*)list_at)[groups - 1].src_tok0 == 16 * (groups - 1) && ((const sk_scatter*)list_at)[groups - 1].count == 16);
    }
    int total = 0, busy = 0;
    for (int i = 1; i <= slots; ++i) { total += recorded[i]; busy += waited[i]; }
    CHECK(total == slots + 5 && busy == 5);         // every long append marked its slot once, whichever way its list went
    CHECK(sk_pool_destroy(p) == SK_OK);
    std::free(d.kv_mem); std::free(d.workspace);
}

// Keys that other sessions hold too are not marked as read by one workgroup alone, and do not count as such: sessions of 32/8 heads of 128 dims,
// 4 KiB a token.
static void check_forks()
{
    sk_pool_desc d = {};
    d.n_q_heads = 32; d.n_kv_heads = 8; d.head_dim = 128; d.max_sessions = 16; d.n_blocks = 1 << 13; d.max_batch_tokens = 1 << 15;
    sk_pool* p = make_pool(d);
    static __attribute__((aligned(16))) char x[16];
    auto grown = [&](int32_t tokens) {
        int32_t id = -1;
        CHECK(sk_session_create(p, &id) == SK_OK && sk_session_append(p, id, nullptr, x, x, tokens, nullptr, SK_F32, nullptr, nullptr) == SK_OK);
        return id;
    };
    auto fork_of = [&](int32_t id, int64_t n) { int32_t f = -1; CHECK(sk_session_fork(p, id, n, &f, nullptr) == SK_OK); return f; };
    auto query_once = [&](int32_t id) {                     // 128 rows per KV head
        launches.clear();
        CHECK(sk_session_query(p, id, x, nullptr, nullptr, 32, x, SK_F32, nullptr, 0, nullptr) == SK_OK);
        CHECK(launches.size() == 1 && launches[0].mode == SK_MODE_REGULAR);
        return launches[0].kv_once;
    };
    auto step_once = [&](const std::vector<int32_t>& ids, int32_t tokens) {      // per item, of a step that queries all of them
        std::vector<int32_t> op(ids.size(), SK_OP_QUERY_A), cu(1, 0), once(ids.size(), -1);
        for (size_t i = 0; i < ids.size(); ++i) cu.push_back(cu.back() + tokens);
        launches.clear(); work.clear();
        CHECK(sk_batch_step(p, (int32_t)ids.size(), ids.data(), op.data(), cu.data(), x, nullptr, nullptr, x, SK_F32, nullptr, nullptr) == SK_OK);
        for (const sk_work& w : work) {
            const size_t i = size_t(w.q_tok0 / tokens);
            CHECK(i < ids.size() && (once[i] < 0 || once[i] == (int32_t)w.once));
            once[i] = (int32_t)w.once;
        }
        return once;
    };
    using flags = std::vector<int32_t>;
    const int32_t a = grown(25000), c = grown(500);
    CHECK(query_once(a) == 1);
    const int32_t b = fork_of(a, 25000);
    CHECK(query_once(a) == 0 && query_once(b) == 0);
    CHECK(step_once({a, b, c}, 16) == (flags{0, 0, 1}));
    // of blocks that go on being shared whatever is evicted and cut off on either side
    CHECK(sk_session_evict_oldest(p, a, 20000, nullptr) == SK_OK);
    CHECK(step_once({a, b, c}, 16) == (flags{0, 0, 1}));
    CHECK(sk_session_truncate(p, b, 20000) == SK_OK);       // b: tokens 0 .. 19,999; a: 20,000 ..
    CHECK(step_once({a, b, c}, 16) == (flags{1, 1, 1}));
    CHECK(sk_session_destroy(p, a) == SK_OK && sk_session_destroy(p, b) == SK_OK);
    // 128-row items, 33 MB each: four sessions of their own are more than 88 MiB, one and three forks of another are not
    std::vector<int32_t> own, forks;
    for (int i = 0; i < 4; ++i) own.push_back(grown(8000));
    CHECK(step_once(own, 32) == (flags{1, 1, 1, 1}));
    for (int i = 0; i < 3; ++i) forks.push_back(fork_of(own[0], 8000));
    CHECK(step_once({forks[0], forks[1], forks[2], own[1]}, 32) == (flags{0, 0, 0, 0}));
    CHECK(step_once({own[1], own[2], own[3], forks[0]}, 32) == (flags{1, 1, 1, 0}));
    for (int32_t f : forks) CHECK(sk_session_destroy(p, f) == SK_OK);
    CHECK(step_once(own, 32) == (flags{1, 1, 1, 1}));
    // an append that is taken back leaves the sessions sharing their last block, which alone they share, as before
    const int32_t e = grown(40), g = fork_of(e, 32);
    CHECK(sk_session_evict_oldest(p, e, 16, nullptr) == SK_OK && sk_session_truncate(p, e, 8) == SK_OK);       // e: the second block, half of it
    CHECK(step_once({e, g}, 16) == (flags{0, 0}));
    const int32_t ids[2] = {e, g}, op[2] = {SK_OP_APPEND, SK_OP_QUERY_A}, cu[3] = {0, 16, 32};
    CHECK(sk_pool_inject_failure(p, SK_SITE_PLAN, 1) == SK_OK);
    CHECK(sk_batch_step(p, 2, ids, op, cu, x, x, x, x, SK_F32, nullptr, nullptr) == SK_E_WORKSPACE);
    CHECK(step_once({e, g}, 16) == (flags{0, 0}));
    drop_pool(p, d);
}

// Pieces of head_dim 64 plans are not kept long for the sake of lists below 16 KiB, which need no copy beyond it either: a step of four
// sessions of 32/8 heads, 83 tokens each behind 1,950, and 17 questions of 16 tokens behind 2,701.
static void check_pieces()
{
    sk_pool_desc d = {};
    d.n_q_heads = 32; d.n_kv_heads = 8; d.head_dim = 64; d.max_sessions = 4; d.n_blocks = 800;
    sk_pool* p = make_pool(d);
    static __attribute__((aligned(16))) char x[16];
    int32_t ids[4], op[4], cu[5] = {0, 83, 166, 249, 332};
    for (int i = 0; i < 4; ++i) {
        op[i] = SK_OP_APPEND;
        CHECK(sk_session_create(p, &ids[i]) == SK_OK && sk_session_append(p, ids[i], nullptr, x, x, i ? 1950 : 2701, nullptr, SK_F32, nullptr, nullptr) == SK_OK);
    }
    work.clear();
    CHECK(sk_session_query_shared_prefix(p, ids[0], nullptr, nullptr, nullptr, 0, x, x, x, 17, 16, nullptr, x, SK_F32, nullptr, nullptr, nullptr) == SK_OK);
    CHECK(work.size() * sizeof(sk_work) > 16384);
    CHECK(sk_session_truncate(p, ids[0], 1950) == SK_OK);
    work.clear();
    CHECK(sk_batch_step(p, 4, ids, op, cu, x, x, x, x, SK_F32, nullptr, nullptr) == SK_OK);
    CHECK(work.size() * sizeof(sk_work) > 16384);
    drop_pool(p, d);
}

// Which short calls merge their parts in the attention launch: by the turns of 1,024 floats that their rows are, and by the parts.
static void check_merges()
{
    static __attribute__((aligned(16))) char x[16];
    auto merged = [&](int dtype, int hq, int hkv, int dim, int32_t n, int32_t tokens, int parts, int32_t splits = 0) {
        sk_pool_desc d = {};
        d.n_q_heads = hq; d.n_kv_heads = hkv; d.head_dim = dim; d.max_sessions = 1; d.n_blocks = n / 16 + 8; d.max_batch_tokens = 16384;
        sk_pool* p = make_pool(d, dtype);
        int32_t id;
        CHECK(sk_session_create(p, &id) == SK_OK && sk_session_append(p, id, nullptr, x, x, n, nullptr, SK_F32, nullptr, nullptr) == SK_OK);
        launches.clear();
        CHECK(sk_session_query(p, id, x, nullptr, nullptr, tokens, x, SK_F32, nullptr, splits, nullptr) == SK_OK);
        CHECK(launches.size() == 1 && launches[0].n_splits == parts);
        const int fuse = launches[0].fuse;
        drop_pool(p, d);
        return fuse;
    };
    CHECK(merged(SK_BF16, 32, 8, 128, 14800, 1, 29) && merged(SK_BF16, 32, 8, 128, 4096, 2, 32));        // one turn
    CHECK(merged(SK_BF16, 32, 8, 128, 4096, 2, 64, 64) && !merged(SK_BF16, 32, 8, 128, 4160, 2, 65, 65));
    CHECK(merged(SK_BF16, 32, 8, 128, 2048, 4, 16) && !merged(SK_BF16, 32, 8, 128, 2049, 4, 17));        // two
    CHECK(merged(SK_BF16, 8, 8, 128, 2048, 9, 16) && !merged(SK_BF16, 8, 8, 128, 2600, 9, 21));
    CHECK(!merged(SK_BF16, 32, 8, 128, 600, 5, 5) && !merged(SK_BF16, 32, 8, 128, 2048, 8, 16));         // three and four
    CHECK(merged(SK_BF16, 32, 8, 128, 512, 8, 4) && !merged(SK_BF16, 32, 8, 128, 513, 8, 5) && merged(SK_BF16, 32, 1, 128, 300, 1, 3));
    CHECK(merged(SK_BF16, 32, 8, 64, 6144, 8, 24) && !merged(SK_BF16, 32, 8, 64, 6145, 8, 25) && merged(SK_BF16, 32, 8, 64, 14800, 4, 29));
    CHECK(!merged(SK_BF16, 12, 4, 128, 6500, 9, 26) && !merged(SK_BF16, 12, 4, 128, 9001, 1, 36));        // KV heads that are no multiple of 8
    CHECK(merged(SK_F32, 4, 4, 64, 3072, 16, 48) && !merged(SK_F32, 4, 4, 64, 3088, 16, 49) && merged(SK_F32, 4, 4, 64, 4096, 4, 64));
    CHECK(merged(SK_F32, 8, 2, 128, 1024, 4, 16) && !merged(SK_F32, 8, 2, 128, 2048, 4, 32) && merged(SK_F32, 8, 2, 128, 2048, 1, 32));
}

// The lists of batched calls: where they are read, that they arrive as they were built, and that a slot of the ring is not
// written again before the kernels that read it are done.
static void check_lists()
{
    static __attribute__((aligned(16))) char x[16];
    sk_pool_desc d = {};
    d.n_q_heads = 4; d.n_kv_heads = 2; d.head_dim = 128; d.max_sessions = 64; d.n_blocks = 1 << 13; d.max_batch_tokens = 1 << 13;
    n_events = 0; std::memset(recorded, 0, sizeof recorded); std::memset(waited, 0, sizeof waited);
    sk_pool* p = make_pool(d);
    const int slots = n_events;
    const char *ws = (const char*)d.workspace, *ring = (const char*)p->ring;
    std::vector<int32_t> ids;
    for (int i = 0; i < 64; ++i) {
        int32_t id;
        CHECK(sk_session_create(p, &id) == SK_OK && sk_session_append(p, id, nullptr, x, x, 1000 + 8 * i, nullptr, SK_F32, nullptr, nullptr) == SK_OK);
        ids.push_back(id);
    }
    std::memset(recorded, 0, sizeof recorded); std::memset(waited, 0, sizeof waited); p->ring_next = 0; std::memset(p->ring_used, 0, sizeof p->ring_used);
    int calls = 0;
    // a step that queries the first n sessions, 40 tokens each; its lists' bytes
    auto step = [&](int n, int kind, bool copied) {
        std::vector<int32_t> op((size_t)n, kind), cu(1, 0);
        for (int i = 0; i < n; ++i) cu.push_back(cu.back() + 40);
        const int before = copies;
        work.clear(); merges.clear(); launches.clear(); list_at = nullptr;
        std::memset((char*)d.workspace + p->L.off_meta, 0xee, p->L.meta_bytes);
        CHECK(sk_batch_step(p, n, ids.data(), op.data(), cu.data(), x, x, x, x, SK_F32, nullptr, nullptr) == SK_OK);
        ++calls;
        CHECK(copies - before == (copied ? 1 : 0));
        const bool scattered = kind == SK_OP_QUERY_B, in_place = !copied;
        if (scattered || in_place) {
            const char* at = (const char*)list_at;
            if (in_place) CHECK(at >= ring && at < ring + slots * p->L.meta_bytes);
            else CHECK(at >= ws + p->L.off_meta && at < ws + p->L.off_meta + p->L.meta_bytes);
        }
        // every session's cached keys once for each KV head, parts as the combine kernel is told
        std::vector<int64_t> keys((size_t)n, 0);
        std::vector<int32_t> parts((size_t)n, 0), told((size_t)n, 1);
        for (const sk_work& w : work) {
            const size_t i = size_t(w.q_tok0 / 40);
            CHECK(i < (size_t)n && w.n_tok == 40 && w.tbl_off == ids[i] * (int32_t)p->L.max_blocks_per_session && w.kv_begin <= w.kv_end);
            if (w.kv_head == 0) { keys[i] += w.kv_end - w.kv_begin; ++parts[i]; }
        }
        for (const sk_comb& c : merges) told[size_t(c.q_tok0 / 40)] = c.n_parts;
        for (int i = 0; i < n; ++i) CHECK(keys[(size_t)i] == 1000 + 8 * i && parts[(size_t)i] == told[(size_t)i]);
        return align_up(work.size() * sizeof(sk_work), 256) + align_up(merges.size() * sizeof(sk_comb), 256) +
               (scattered ? align_up((size_t)n * 3 * sizeof(sk_scatter), 256) : 0);
    };
    CHECK(step(4, SK_OP_QUERY_B, true) <= 16384 && step(4, SK_OP_QUERY_A, true) <= 16384);
    CHECK(step(64, SK_OP_QUERY_A, false) > 16384);                  // nothing to scatter: a launch of copies alone
    const size_t bytes = step(64, SK_OP_QUERY_B, false);
    int total = 0, busy = 0;
    for (int i = 1; i <= slots; ++i) { total += recorded[i]; busy += waited[i]; }
    CHECK(total == calls && busy == std::max(0, calls - slots));
    step(64, SK_OP_QUERY_B, false);
    CHECK(waited[(calls - 1) % slots + 1] == (calls > slots ? 1 : 0));
    // a list region that holds the lists, but not the copies' items beside them: one copy
    const size_t meta = p->L.meta_bytes;
    p->L.meta_bytes = bytes;
    CHECK(step(64, SK_OP_QUERY_B, true) == bytes);
    p->L.meta_bytes = meta;
    // a launch that reports an error is on the stream all the same: its slot stays busy, no session is changed
    launch_error = (int)hipErrorInvalidValue;
    const int slot = p->ring_next, marks = recorded[slot + 1];
    std::vector<int32_t> op(64, SK_OP_QUERY_B), cu(1, 0);
    for (int i = 0; i < 64; ++i) cu.push_back(cu.back() + 40);
    CHECK(sk_batch_step(p, 64, ids.data(), op.data(), cu.data(), x, x, x, x, SK_F32, nullptr, nullptr) == SK_E_HIP && recorded[slot + 1] == marks + 1);
    drop_pool(p, d);

    // up to 8,192 groups of 16 tokens a batched call's scatter list is read where it lies, a longer one behind a copy of all lists
    sk_pool_desc e = {};
    e.n_q_heads = e.n_kv_heads = 1; e.head_dim = 64; e.max_sessions = 1; e.n_blocks = 1 << 14; e.max_batch_tokens = 1 << 18;
    p = make_pool(e);
    int32_t id;
    CHECK(sk_session_create(p, &id) == SK_OK);
    for (int32_t groups : {8192, 8193}) {
        const int32_t what = SK_OP_APPEND, ends[2] = {0, 16 * groups};
        const int before = copies;
        work.clear();
        CHECK(sk_batch_step(p, 1, &id, &what, ends, x, x, x, x, SK_F32, nullptr, nullptr) == SK_OK && copies - before == (groups > 8192 ? 1 : 0));
        CHECK(((const sk_scatter*)list_at)[groups - 1].src_tok0 == 16 * (groups - 1));
        int64_t rows = 0;
        for (const sk_work& w : work) if (w.kv_begin == 0) rows += w.n_tok;
        CHECK(rows == 16 * groups && sk_session_truncate(p, id, 0) == SK_OK);
    }
    drop_pool(p, e);
}

int main(int argc, char** argv)
{
    const char* what = argc > 1 ? argv[1] : "ring";
    if (!std::strcmp(what, "ring")) check_ring();
    else if (!std::strcmp(what, "forks")) check_forks();
    else if (!std::strcmp(what, "pieces")) check_pieces();
    else if (!std::strcmp(what, "merges")) check_merges();
    else if (!std::strcmp(what, "lists")) check_lists();
    else return 1;
    std::printf("fake device ok\n");
    return 0;
}
