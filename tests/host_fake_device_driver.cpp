// The library's host code against a device that is not there: the HIP calls and the kernel launchers are replaced by functions
// that count, so that what a call asks the runtime for can be checked where no GPU is.  Built and run by
// tests/test_host_fake_device.py; exits non-zero on a mismatch.
#include <hip/hip_runtime_api.h>

#include <cstdio>
#include <cstdlib>
#include <cstring>

#include "../include/sk.h"
#include "../paper_2605_13784_amd/csrc/sk_internal.h"

#define CHECK(c) do { if (!(c)) { std::fprintf(stderr, "check failed at line %d: %s\n", __LINE__, #c); std::exit(1); } } while (0)

static int n_events, recorded[16], waited[16], copies, launch_error;
static unsigned host_flags;
static const void* list_at;

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
int sk_launch_scatter(const sk_geom&, const void*, const void*, const sk_scatter* items, int32_t, int32_t*, unsigned char*, unsigned char*, void*)
{
    list_at = items;
    const int e = launch_error;
    launch_error = 0;
    return e;
}
int sk_launch_scatter_args(const sk_geom&, const void*, const void*, const sk_scatter_list&, int32_t, int32_t*, unsigned char*, unsigned char*, void*) { return 0; }
int sk_launch_attention(const sk_launch&, int, int32_t, void*, void*, void*) { return 0; }
int sk_launch_attention_small(const sk_launch&, const sk_commit&, int32_t, void*, void*, void*) { return 0; }
int sk_launch_combine(const sk_launch&, int32_t, int32_t, int64_t, void*, void*, void*) { return 0; }
int sk_launch_gather(const sk_geom&, int32_t, int64_t, int64_t, void*, void*, void*) { return 0; }
int sk_launch_copy_block(const sk_geom&, unsigned char*, int32_t, int32_t, void*) { return 0; }

int main()
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
    std::printf("fake device ok\n");
    return 0;
}
