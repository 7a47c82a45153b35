// Host side of the library: pool bookkeeping (free list, sessions, block tables), argument
// checks, the planner that cuts a call into workgroups, and the C ABI of include/sk.h.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdlib>
#include <cstring>
#include <deque>
#include <new>
#include <vector>

#include "../../include/sk.h"
#include "sk_internal.h"

namespace {

thread_local int g_last_hip = 0;

constexpr int kRingSlots = 4;
constexpr size_t kMinMetaBytes = 4u << 20;       // least size of the device region for uploaded lists (= ring slot size)
constexpr int kPartSlotRows = 128;               // rows reserved per partial slot
constexpr int kDefaultTargetWgs = 512;
constexpr int kDefaultWaitPolls = 256;           // polls a workgroup waits for the others of its unit (about 1 us each)

inline size_t align_up(size_t x, size_t a) { return (x + a - 1) / a * a; }
inline int ilog2_exact(int64_t x) { int l = 0; while ((int64_t(1) << l) < x) ++l; return ((int64_t(1) << l) == x) ? l : -1; }

// A session's tokens live at *storage indices* 0 .. len-1; block i of `blocks` holds storage
// indices i*B .. i*B+B-1.  Storage indices [frozen, win) are evicted (Region-1 FIFO eviction behind
// a frozen Region 0): what the session holds is [0, frozen) followed by [win, len).  Whole blocks
// inside the hole are returned to the pool and the storage indices behind them shifted down, so
// the hole always spans less than two blocks; what is left of it is masked in the kernels.
struct Session {
    bool live = false;
    int64_t len = 0;
    int64_t frozen = 0, win = 0;
    std::vector<int32_t> blocks;
    mutable bool may_share = false;      // forked, or a fork: other sessions may hold some of its blocks too (holds_shared)
    int64_t retained() const { return frozen + (len - win); }
};

struct Layout {
    int elem = 0, G = 0;
    int64_t head_stride = 0, blk_stride = 0, v_off = 0;
    int64_t eph_head_stride = 0, eph_blk_stride = 0, eph_v_off = 0;
    int64_t max_blocks_per_session = 0, max_session_tokens = 0;
    int32_t max_batch_tokens = 0;
    int64_t eph_blocks = 0;
    int64_t part_slots = 0;
    int64_t sync_units = 0;           // 8-byte merge counters (a pair of 32-bit ones, or a sixteenth of a line)
    size_t meta_bytes = 0;            // device region for uploaded lists; also the size of a pinned ring slot
    size_t kv_bytes = 0;
    // workspace offsets
    size_t off_tables = 0, off_ident = 0, off_meta = 0, off_sync = 0, off_part_ml = 0, off_part_o = 0, off_eph = 0, ws_bytes = 0;
};

bool derive_layout(const sk_pool_desc& d, Layout& L)
{
    if (d.dtype != SK_F32 && d.dtype != SK_BF16) return false;
    if (d.n_kv_heads <= 0 || d.n_q_heads <= 0 || d.n_q_heads % d.n_kv_heads) return false;
    if (d.head_dim != 64 && d.head_dim != 128) return false;
    if (d.block_tokens < 16 || d.block_tokens > 1024 || ilog2_exact(d.block_tokens) < 0) return false;
    if (d.n_blocks <= 0 || d.n_blocks > (int64_t(1) << 30) || d.max_sessions <= 0 || d.max_sessions > (1 << 20)) return false;
    if (d.max_session_tokens < 0 || d.max_batch_tokens < 0) return false;
    L.elem = d.dtype == SK_F32 ? 4 : 2;
    L.G = d.n_q_heads / d.n_kv_heads;
    L.v_off = int64_t(d.block_tokens) * d.head_dim * L.elem;
    // [kv_head][block][K | V]: the blocks of one head are contiguous, so a workgroup (which
    // streams one head) reads whole consecutive 8 KiB pieces when the table is in order
    L.blk_stride = 2 * L.v_off;
    L.head_stride = L.blk_stride * d.n_blocks;
    L.eph_v_off = int64_t(16) * d.head_dim * L.elem;
    L.eph_blk_stride = 2 * L.eph_v_off;
    L.eph_head_stride = 0;     // set once the number of staging blocks is known
    int64_t mst = d.max_session_tokens ? d.max_session_tokens : d.n_blocks * d.block_tokens;
    mst = std::min<int64_t>(mst, d.n_blocks * d.block_tokens);
    mst = std::min<int64_t>(mst, int64_t(kMinMetaBytes / 4) * d.block_tokens);    // a session's block table is uploaded in one piece
    if (mst > (int64_t(1) << 29)) return false;       // positions are int32 with head room
    L.max_session_tokens = mst;
    L.max_blocks_per_session = (mst + d.block_tokens - 1) / d.block_tokens;
    // offsets into the device block tables are 32-bit
    if (int64_t(d.max_sessions) * L.max_blocks_per_session >= (int64_t(1) << 31)) return false;
    L.max_batch_tokens = d.max_batch_tokens ? d.max_batch_tokens : 4096;
    if (L.max_batch_tokens > (1 << 20)) return false;
    {   // The lists a batched call uploads always fit when every row tile is one workgroup per KV head
        // (the planner falls back to that): a call has at most max_batch_tokens tokens in at most
        // min(max_sessions, max_batch_tokens) items (question batches: one tile per question at worst),
        // so at most tiles_max row tiles and scat_max 16-token scatter groups.
        const int64_t items_max = std::min<int64_t>(std::max(d.max_sessions, 1024), L.max_batch_tokens);
        const int64_t tpt_min = std::max(1, 16 / L.G);                          // tokens per row tile of the smallest kernel
        const int64_t tiles_max = L.max_batch_tokens / tpt_min + items_max;
        const int64_t scat_max = L.max_batch_tokens / 16 + 2 * items_max + 2;
        const int64_t need = tiles_max * d.n_kv_heads * int64_t(sizeof(sk_work) + sizeof(sk_comb)) + scat_max * int64_t(sizeof(sk_scatter)) + 16 * 256;
        // Capped at 64 MiB: a step whose lists do not fit even then is refused with SK_E_WORKSPACE and
        // leaves every session as it was.
        L.meta_bytes = align_up(std::max<size_t>(kMinMetaBytes, std::min<size_t>(size_t(need), size_t(64) << 20)), 256);
    }
    L.eph_blocks = (L.max_batch_tokens + 15) / 16 + std::max(d.max_sessions, 1024) + 1;
    L.eph_head_stride = L.eph_blk_stride * L.eph_blocks;
    int64_t rows = int64_t(L.max_batch_tokens) * d.n_q_heads;
    L.part_slots = 2048 + 2 * ((rows + kPartSlotRows - 1) / kPartSlotRows);
    L.kv_bytes = size_t(2 * L.v_off) * size_t(d.n_kv_heads) * size_t(d.n_blocks);
    size_t off = 0;
    L.off_tables = off; off = align_up(off + size_t(d.max_sessions) * L.max_blocks_per_session * 4, 256);
    L.off_ident = off;  off = align_up(off + size_t(L.eph_blocks) * 4, 256);
    L.off_meta = off;   off = align_up(off + L.meta_bytes, 256);
    // Merge counters: a pair per (row tile, KV head) of a call of the ring kernels, whose tiles have at least 64 rows; for the
    // kernels with one 128-byte line per unit the planners check that their units fit
    L.sync_units = (rows / 64 + std::max(d.max_sessions, 1024) + 2) * d.n_kv_heads;
    L.off_sync = off;   off = align_up(off + size_t(L.sync_units) * 8, 256);
    L.off_part_ml = off; off = align_up(off + size_t(L.part_slots) * kPartSlotRows * 4 * 4, 256);
    L.off_part_o = off; off = align_up(off + size_t(L.part_slots) * kPartSlotRows * d.head_dim * 4, 256);
    L.off_eph = off;    off = align_up(off + size_t(L.eph_blocks) * L.eph_blk_stride * d.n_kv_heads, 256);
    L.ws_bytes = off;
    return true;
}

}  // namespace

struct sk_pool {
    sk_pool_desc d;
    Layout L;
    bool device = false;
    std::deque<int32_t> free_blocks;
    std::vector<Session> sessions;
    std::vector<int32_t> free_ids;
    int64_t blocks_in_use = 0;
    std::vector<int32_t> refcnt;         // sessions holding each block (forks share the blocks of a prefix)
    // pinned staging ring for uploaded lists
    unsigned char* ring = nullptr;
    hipEvent_t ring_ev[kRingSlots] = {};
    bool ring_used[kRingSlots] = {};
    int ring_next = 0;
    sk_geom geom;
    sk_pool_stats stats = {};
    sk_launch_info last = {};
    // Tuning switches, read from the environment once when the pool is created (see sk_pool_create).
    int target_wgs = kDefaultTargetWgs;
    bool target_wgs_set = false;
    bool force_simple = false, no_small = false, no_256 = false, no_pack = false, no_interleave = false, no_stream_loads = false;
    int distrust = 0;                    // SK_SMALL_DISTRUST (tests)
    bool p128 = true;                    // SK_NO_P128=1: never the eight-wave 128-row instance
    int64_t p128_min_tokens = -1;        // SK_P128_MIN_TOKENS: cached tokens from which it is taken; -1: by the keys of a workgroup (kP128MinKeys)
    int64_t stream_min_tokens = -1;      // SK_STREAM_MIN_TOKENS: cached tokens from which the 128-row instances load non-temporal; -1: by the bytes of K/V (streams_once)
    bool fuse = false;                   // SK_FUSE=1: single-session calls merge their split partials inside the attention kernel
    bool fuse_list = false;              // batched calls too (the last workgroup of a unit merges alone)
    bool merge_fences = false;           // SK_MERGE_FENCES=1: full fences around the arrival (for comparison)
    int wait_polls = kDefaultWaitPolls;
    int n_cus = 256;                     // compute units of the device the pool was created on
    // test hook (sk_pool_inject_failure): the countdown-th arrival at `inject_site` fails
    int inject_site = 0, inject_countdown = 0;
    // optional kernel timing
    bool profiling = false;
    struct ProfRec { hipEvent_t start, stop; int32_t call, kind; };   // one kernel dispatch; kind 0 attention, 1 combine
    std::vector<ProfRec> prof;           // records (events are created once and reused)
    size_t prof_used = 0;                // records in use
    int32_t prof_calls = 0;              // calls since the last read
};

namespace {

#define SK_HIP(expr)                                        \
    do {                                                    \
        hipError_t e_ = (expr);                             \
        if (e_ != hipSuccess) { g_last_hip = (int)e_; return SK_E_HIP; } \
    } while (0)

bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15) == 0; }

Session* get_session(sk_pool* p, int32_t id)
{
    if (!p || id < 0 || id >= (int32_t)p->sessions.size() || !p->sessions[id].live) return nullptr;
    return &p->sessions[id];
}
const Session* get_session(const sk_pool* p, int32_t id) { return get_session(const_cast<sk_pool*>(p), id); }

int64_t blocks_needed(const sk_pool* p, int64_t len, int64_t add)
{
    const int64_t B = p->d.block_tokens;
    return (len + add + B - 1) / B - (len + B - 1) / B;
}

// Whether another session holds one of the session's blocks too (forks share those of their prefix, and evictions
// and truncations on either side can leave any of them shared).  Blocks come to be shared by a fork alone, so that a session found to
// hold none is not looked at again before the next.
bool holds_shared(const sk_pool* p, const Session& s)
{
    if (!s.may_share) return false;
    for (int32_t b : s.blocks)
        if (p->refcnt[(size_t)b] > 1) return true;
    s.may_share = false;
    return false;
}

// Test hook: true when a failure was ordered for this site and its countdown has run out.  The sites
// are visited in the same order by device pools and by metadata-only pools (which skip the HIP call
// itself), so the error paths behind them can be exercised without a GPU.
bool inject(sk_pool* p, int site)
{
    if (p->inject_site != site || p->inject_site == 0) return false;
    if (--p->inject_countdown > 0) return false;
    p->inject_site = 0;
    g_last_hip = (int)hipErrorUnknown;
    return true;
}

// Takes a ring slot (waiting for the copy that last used it), returns its host pointer (null for a
// metadata-only pool).  Changes nothing when it fails.
int ring_acquire(sk_pool* p, int* slot, unsigned char** host)
{
    if (inject(p, SK_SITE_RING)) return SK_E_HIP;
    *slot = 0; *host = nullptr;
    if (!p->device) return SK_OK;
    int s = p->ring_next;
    if (p->ring_used[s]) SK_HIP(hipEventSynchronize(p->ring_ev[s]));
    p->ring_next = (s + 1) % kRingSlots;
    *slot = s;
    *host = p->ring + size_t(s) * p->L.meta_bytes;
    return SK_OK;
}

// Marks ring slot `slot` busy until what the stream holds now, which reads it, is done.
void ring_busy(sk_pool* p, int slot, hipStream_t st)
{
    if (hipEventRecord(p->ring_ev[slot], st) != hipSuccess) (void)hipStreamSynchronize(st);   // the slot is free either way
    p->ring_used[slot] = true;
}

// Copies `bytes` from ring slot `slot` to `dev` on the stream and marks the slot busy until then.
int ring_copy(sk_pool* p, int slot, void* dev, size_t bytes, hipStream_t st)
{
    if (inject(p, SK_SITE_UPLOAD)) return SK_E_HIP;
    if (!p->device) return SK_OK;
    SK_HIP(hipMemcpyAsync(dev, p->ring + size_t(slot) * p->L.meta_bytes, bytes, hipMemcpyHostToDevice, st));
    ring_busy(p, slot, st);
    return SK_OK;
}

int ring_upload(sk_pool* p, int slot, size_t bytes, hipStream_t st)
{
    return ring_copy(p, slot, p->device ? (unsigned char*)p->d.workspace + p->L.off_meta : nullptr, bytes, st);
}

// With profiling on: a call announces itself (prof_call) and asks for a pair of events per kernel
// it launches (prof_pair); the launchers hand them to the runtime, which stamps them with the
// dispatch's own start and end times.
constexpr size_t kProfMax = 4 * 4096;
int32_t prof_call(sk_pool* p) { return p->profiling ? p->prof_calls++ : -1; }
bool prof_pair(sk_pool* p, int32_t call, int32_t kind, void** start, void** stop)
{
    *start = *stop = nullptr;
    if (call < 0 || p->prof_used >= kProfMax) return false;
    if (p->prof.size() <= p->prof_used) {
        sk_pool::ProfRec r = {};
        if (hipEventCreate(&r.start) != hipSuccess) return false;
        if (hipEventCreate(&r.stop) != hipSuccess) { (void)hipEventDestroy(r.start); return false; }
        p->prof.push_back(r);
    }
    sk_pool::ProfRec& r = p->prof[p->prof_used++];
    r.call = call; r.kind = kind;
    *start = r.start; *stop = r.stop;
    return true;
}

// Which attention kernel takes a tile of `max_rows` query rows per KV head.
struct Variant { int id; int rows_per_slot; int tok_per_tile; };

// `allow_256`: the caller can launch the 256-row tile, whose eight waves and key ring (128 KiB, 64 at head_dim 64) take a CU alone.
// `cached` >= 0: a single-session call over so many cached tokens, which may take the kernel for at most 32 rows.  Up to
// 128 MiB of cached K/V, where the ring kernel's stream gets close (us per cache-only query in a stream of them, ring and combine
// kernel -> this one, one query token / 32 rows):
//   heads         2,600 cached              9,001                     32,768                    65,536                    131,072
//   32/8  d 128   11.9 ->  6.3/12.0 ->  9.7 15.2 ->  9.4/15.2 -> 12.5 29.3 -> 23.0/29.4 -> 25.4 -                         -
//   28/4  d 128   11.7 ->  6.8/11.8 ->  9.3 13.9 ->  9.9/13.8 -> 11.4 20.0 -> 15.5/19.9 -> 16.9 29.7 -> 25.4/29.7 -> 26.7 -
//    8/1  d 128   11.4 ->  6.8/11.7 ->  9.2 13.2 -> 10.0/13.5 -> 11.3 16.2 -> 12.1/16.4 -> 13.8 21.4 -> 17.2/22.2 -> 19.2 27.0 -> 20.6/27.2 -> 22.3
//   24/12 d 128   11.6 ->  6.7/12.1 ->  9.9 17.5 -> 12.7/17.7 -> 14.9 -                         -                         -
//   14/2  d 64     9.2 ->  5.5/ 9.5 ->  7.9 10.4 ->  6.5/10.8 ->  9.0 13.1 ->  9.6/13.5 -> 10.2 18.3 -> 12.7/18.3 -> 13.3 22.9 -> 16.5/23.3 -> 17.4
//   32/8  d 64     9.4 ->  5.2/ 9.5 ->  8.1 11.1 ->  6.4/11.2 ->  9.0 17.2 -> 13.8/17.4 -> 15.1 26.6 -> 22.9/27.1 -> 24.3 -
// (beyond, before short queries' first loads and merge were what they are: 32/8 of 128 dims at 131,072 90.2 -> 96.8)
constexpr int64_t kSmallMaxBytes = int64_t(128) << 20;
constexpr int64_t kP128MinKeys = 512;         // keys of a workgroup from which the 128-row tile takes eight waves (plan_regular)
bool pick_variant(const sk_pool* p, int64_t n_tok, Variant& v, bool allow_256 = false, int64_t cached = -1)
{
    const int G = p->L.G;
    // any group size up to 128 (multi-query models): a tile holds floor(rows / G) tokens, at least one
    const bool mfma_ok = p->d.dtype == SK_BF16 && (p->d.head_dim == 128 || p->d.head_dim == 64) && G <= 128;
    if (mfma_ok && !p->force_simple) {
        if (cached >= 0 && !p->no_small && n_tok * G <= 32 && cached * p->d.n_kv_heads * p->d.head_dim * 4 <= kSmallMaxBytes) { v.id = SK_KV_SMALL; v.rows_per_slot = 32; v.tok_per_tile = 32 / G; }
        else if (allow_256 && n_tok * G > 128) { v.id = SK_KV_MFMA256; v.rows_per_slot = 256; v.tok_per_tile = 256 / G; }
        else if (n_tok * G > 64 || G > 64) { v.id = SK_KV_MFMA128; v.rows_per_slot = 128; v.tok_per_tile = 128 / G; }
        else { v.id = SK_KV_MFMA64; v.rows_per_slot = 64; v.tok_per_tile = 64 / G; }
        return true;
    }
    if (G > 16) return false;
    v.id = SK_KV_SIMPLE; v.rows_per_slot = 16; v.tok_per_tile = std::max(1, 16 / G);
    return true;
}

void fill_launch_common(const sk_pool* p, sk_launch& L, const void* q, void* out, int out_dtype, float* lse, const Variant& v)
{
    memset(&L, 0, sizeof L);
    L.g = p->geom;
    L.q = q; L.out = out; L.lse = lse;
    unsigned char* ws = (unsigned char*)p->d.workspace;
    L.part_ml = (float*)(ws + p->L.off_part_ml);
    L.part_o = (float*)(ws + p->L.off_part_o);
    L.sync = (uint32_t*)(ws + p->L.off_sync);
    L.out_dtype = out_dtype == SK_F32 ? 0 : 1;
    L.rows_per_slot = v.rows_per_slot;
}

// Regular-mode attention over one session: n_tok new tokens at positions pos0.. (or no causal
// limit), kv_len cached tokens, optionally one uncommitted segment already in staging block 0.
// plan_regular decides the decomposition and is the only part that can refuse the call (it reads
// nothing but sizes, so it runs before a call changes anything); launch_regular enqueues it.
struct RegPlan {
    Variant v;
    sk_launch L;           // everything but the pointers
    int32_t wgs = 0, base_wgs = 0, parts = 1;
    int64_t kv_len = 0;
    const void *own_k = nullptr, *own_v = nullptr;     // SMALL: the call's own K/V
    sk_commit commit;                                  // SMALL: what an append commits in the same launch
    int32_t commit_items = 0;
    bool enqueued = false;                             // set by launch_regular once the attention kernel is on the stream
};

// Whether the last workgroup of a unit merges its parts, `rows` rows each, instead of the combine kernel in a second launch.  Its lanes
// take a turn for every 1,024 floats of the rows, one behind the other: two round trips to the L2 for up to 16 parts, one more for every 16
// further ones.  The combine kernel does all of them at once, behind a launch of about 1 us of the device's time.  us per query, combine
// kernel -> merged in the launch, in a stream of queries / alone (a wait behind each), 32/8 heads:
//   rows (turns) d 128   5 parts [600 cached]         16 [2,048]                   21 [2,600]                   32 [32,768]
//    8  (1)              7.9 -> 6.0/19.4 -> 18.7      7.6 -> 5.9/19.5 -> 18.7      7.5 -> 6.3/19.9 -> 19.0      24.4 -> 23.4/36.4 -> 35.5
//   12  (2)              8.0 -> 6.9/19.7 -> 19.6      7.7 -> 6.9/19.7 -> 19.6      8.0 -> 8.0/20.2 -> 20.3      24.9 -> 25.3/37.0 -> 37.6
//   16  (2)              7.9 -> 7.2/19.8 -> 20.1      7.8 -> 7.3/20.0 -> 20.1      8.1 -> 8.6/20.4 -> 20.9      25.2 -> 25.9/37.2 -> 38.2
//   20  (3)              7.8 -> 8.1/20.1 -> 20.9      8.1 -> 8.4/20.2 -> 20.9      8.4 -> 9.8/20.7 -> 22.1      25.4 -> 27.3/37.6 -> 39.7
//   32  (4)              8.0 -> 9.5/20.7 -> 22.2      8.3 -> 9.9/20.8 -> 22.6      8.7 -> 11.8/21.3 -> 24.2     26.1 -> 30.0/38.2 -> 42.3
// Up to four parts are merged whatever the rows: 1.0 us more of the device's time at 32 rows for 1.8 less of the host's (6.2 of 8.0 a call).
// Two turns of 64 dims are merged up to 32 parts where the host's second launch is what a stream waits for (20 rows,
// combine -> merged: 2,600 cached 8.1 -> 7.4/19.6 -> 20.2, 5,000 8.3 -> 7.8/20.3 -> 20.6, 6,500 7.8 -> 7.8/19.4 -> 20.3, 9,001 7.8 -> 8.4, 14,800 9.0 -> 10.1); fp32,
// whose workgroups end further apart, one turn up to 48 (4/4 heads, 8 rows: 2,048 cached, 33 parts 8.4 -> 8.0; 16 rows: 32 parts 8.5 ->
// 8.1, 4,096, 64 parts 9.0 -> 10.0), or 64 where a single wave has all of it (4 rows: 9.0 -> 8.7).
// Offsets of the rounds of sixteen it reads the parts in are 32-bit; at most 64 parts (their weights' place in LDS).
bool can_merge(const sk_pool* p, const Variant& v, int64_t rows, int64_t parts, int64_t kv_len)
{
    const int64_t floats = rows * p->d.head_dim, turns = (floats + 1023) / 1024;
    const int64_t most = turns == 1 ? (p->L.elem == 2 || floats <= 256 ? 64 : 48) : turns == 2 ? (p->d.head_dim == 64 && kv_len <= 6144 ? 32 : 16) : 4;
    const int64_t step = int64_t(p->d.n_kv_heads) * v.rows_per_slot * p->d.head_dim * 4;
    return parts > 1 && parts <= most && (parts + 15) * step < (int64_t(1) << 32);
}

// The kernel for at most 32 rows per KV head: cached tokens in parts of whole 32-key tiles, four waves to a
// part; own_cnt tokens of the call itself (uncommitted, or being appended) behind them.
int plan_small(const sk_pool* p, int64_t kv_len, int32_t own_cnt, int32_t n_splits_req, RegPlan& R)
{
    sk_launch& L = R.L;
    const int64_t Hkv = p->d.n_kv_heads, cap = p->L.part_slots * kPartSlotRows / (Hkv * R.v.rows_per_slot);
    int64_t chunk = 0, parts = 1;
    auto cut = [&](int64_t S) {
        chunk = kv_len > 0 ? (kv_len + S - 1) / S : 64;
        if (n_splits_req <= 0) chunk = std::max<int64_t>((chunk + 127) / 128 * 128, 128);      // a tile for every wave
        chunk = (chunk + 63) / 64 * 64;
        for (;; chunk *= 2) {
            S = (kv_len + chunk - 1) / chunk;
            const int64_t last = kv_len - (S - 1) * chunk;          // keys of the last part
            // the own tokens are a tile of the last part if a wave is free there, else a part of their own
            parts = std::max<int64_t>(1, S + ((own_cnt > 0 && S > 0 && (last + 31) / 32 > 3) ? 1 : 0));
            if (S == 1 && parts == 2 && (n_splits_req == 1 || cap < 2)) parts = 1;      // (or a fifth tile of one workgroup)
            if (parts <= 1 || parts <= cap) break;
        }
    };
    // The last workgroup to finish merges the parts of a KV head (they lie a multiple of 8 workgroups apart, hence on
    // one XCD) if they are few enough for one workgroup to read (can_merge).
    // A head then has the CUs of one XCD.  Where the heads are no multiple of 8, others have less to do or nothing: up to
    // 4 MiB of K/V for the busiest XCD the launch saved is worth more than that (us per query of one token, merged in the
    // launch against by the combine kernel: 8 heads on 1, 5,000 cached tokens 7.5 against 8.8, 8,100 8.0 - 9.2, 9,001 9.3
    // - 9.9, 13,000 11.0 - 10.0, 32,768 18.4 - 12.0; 12 on 4, 6,500 7.1 - 8.4, 9,001 9.1 - 9.1, 13,000 12.1 - 9.4; 24 on
    // 12, 4,096 7.1 - 7.7, 5,000 9.6 - 8.4; 14 on 2 of 64 dims, 14,800 7.5 - 7.8, 18,000 8.8 - 8.1), and the parts are cut for its
    // CUs alone, also where their rows are more than one workgroup merges (12 on 4, 27 rows at 6,500 in 26 parts 10.2, in 51
    // 10.8; at 8,100 in 32 10.3, in 64 10.9).
    // For the combine kernel, which reads the statistics of 64 parts at once, no more than 64 of up to 1,024 keys (8
    // heads on 1: 32,768 tokens in 256 parts 27.9, 128 19.9, 64 16.4, 32 18.3; 65,536 28.9 - 21.3 - 20.7 - 26.9).
    constexpr int64_t kXcds = 8, kOneXcdBytes = int64_t(4) << 20;
    const int64_t wanted = std::max<int64_t>(1, (p->target_wgs_set ? p->target_wgs : p->n_cus) / Hkv);
    const int64_t heads_per_xcd = (Hkv + kXcds - 1) / kXcds;
    const bool even = Hkv % kXcds == 0;
    if (even || kv_len * heads_per_xcd * p->d.head_dim * 4 <= kOneXcdBytes) {
        cut(n_splits_req > 0 ? n_splits_req : even ? wanted : std::min(wanted, std::max<int64_t>(1, p->n_cus / kXcds / heads_per_xcd)));
        L.fuse = (can_merge(p, R.v, int64_t(L.n_tok) * p->L.G, parts, kv_len) && Hkv * 16 <= p->L.sync_units) ? 1 : 0;
    }
    else cut(n_splits_req > 0 ? n_splits_req : std::min(wanted, std::max<int64_t>(64, kv_len / 1024)));
    L.chunk = (int32_t)chunk; L.n_splits = (int32_t)parts;
    L.own_cnt = own_cnt; L.own_mode = SK_OWN_SMALL;
    L.head_pad = L.fuse ? (int32_t)((Hkv + 7) / 8 * 8) : (int32_t)Hkv;
    L.by_pad = sk_make_div((uint32_t)L.head_pad);
    L.distrust = p->distrust;
    R.base_wgs = (int32_t)Hkv; R.parts = (int32_t)parts; R.wgs = int32_t(L.head_pad * parts); R.kv_len = kv_len;
    return SK_OK;
}

// fp32 pools: keys are the cached tokens, padded to whole 16-key tiles, then the call's own; parts of at least 64 keys
// (a tile for each of the four waves).
int plan_f32(const sk_pool* p, int64_t kv_len, int32_t own_cnt, int32_t n_splits_req, RegPlan& R)
{
    sk_launch& L = R.L;
    const int64_t Hkv = p->d.n_kv_heads, units = L.n_tiles * Hkv, cap = p->L.part_slots * kPartSlotRows / (units * R.v.rows_per_slot);
    const int64_t keys = (kv_len + 15) / 16 * 16 + own_cnt;
    const int64_t S = n_splits_req > 0 ? n_splits_req : std::max<int64_t>(1, (p->target_wgs + units / 2) / units);
    int64_t chunk = std::max<int64_t>(64, ((keys + S - 1) / S + 63) / 64 * 64), parts;
    for (;; chunk *= 2) {
        parts = std::max<int64_t>(1, (keys + chunk - 1) / chunk);
        if (parts <= 1 || parts <= cap) break;
    }
    L.chunk = (int32_t)chunk; L.n_splits = (int32_t)parts; L.by_chunk = sk_make_div((uint32_t)chunk);
    L.own_cnt = own_cnt; L.own_mode = SK_OWN_F32;
    // Merged by the last workgroup of a unit while that is a few rounds of loads (can_merge).  Few units leave XCDs idle here
    // too, but such calls stay short: 1/1, 16/1, 10/2, 4/4 and 8/2 heads with 1 to 1,024 tokens at 128 to 32,768 cached are 1.4
    // to 17 times as fast as with the fp32-FMA kernel and its combine, none slower.
    L.fuse = (can_merge(p, R.v, std::min<int64_t>(L.n_tok, R.v.tok_per_tile) * p->L.G, parts, kv_len) && units * 16 <= p->L.sync_units) ? 1 : 0;
    const int64_t pad = L.fuse ? (units + 7) / 8 * 8 : units;
    if (pad * parts > (int64_t(1) << 30)) return SK_E_WORKSPACE;
    L.head_pad = (int32_t)pad; L.by_pad = sk_make_div((uint32_t)pad); L.by_tiles = sk_make_div((uint32_t)L.n_tiles);
    L.distrust = p->distrust;
    R.base_wgs = (int32_t)units; R.parts = (int32_t)parts; R.wgs = int32_t(pad * parts); R.kv_len = kv_len;
    return SK_OK;
}

// Whether the 128-row instances load keys that no other workgroup of the launch reads non-temporal.  The default policy costs the keys'
// way into the last-level cache of 256 MiB and pays if they are still there when they are read again, which depends on what the
// program reads in between (a model reads each layer's pool in turn; nobody tells the library) and not on this call.  The line
// is a compromise: where the keys of three sessions or layers, read in turn, push one another out.  Of more in turn, shorter ones
// would gain too; one session read again and again loses above it.  us per query of 32 tokens of 32/8 heads, default -> non-temporal:
//                           one again and again   two in turn      three            eight
//   14,800 cached   61 MB   23.4 -> 23.3          22.2 -> 23.2     22.2 -> 23.2     25.6 -> 23.4
//   18,000          74 MB   24.5 -> 25.5          24.1 -> 25.3     24.4 -> 25.5     28.7 -> 25.4
//   20,000          82 MB   25.7 -> 26.8          25.1 -> 26.6     27.6 -> 26.7     30.3 -> 26.7
//   22,528          92 MB   28.0 -> 29.0          26.4 -> 28.0     30.7 -> 27.9     33.7 -> 28.0
//   25,000         102 MB   28.8 -> 30.6          27.8 -> 30.6     33.1 -> 30.4     36.7 -> 30.3
//   32,768         134 MB   34.0 -> 34.5          35.3 -> 34.9     40.8 -> 34.6     41.1 -> 34.6
//   48,000         197 MB   43.9 -> 47.8          54.3 -> 47.4     54.1 -> 47.6     54.4 -> 47.7
// (kernel alone: 8,000 cached, 33 MB, 12.4 -> 12.6 again and again, 12.5 -> 13.2 of three, 14.4 -> 13.3 of eight in turn; 32,768 25.7 -> 28.4,
// 36.8 -> 29.1, 36.8 -> 29.0)
// The 64-row instance: 10.3 -> 10.5 / 10.9 -> 11.3 / 12.0 -> 11.8 at 8,000 (16 tokens), 23.8 -> 25.4 / 31.8 -> 26.3 / 31.8 -> 26.5 at 32,768.
// The 256-row one: 38.0 -> 41.9 / 46.3 -> 44.5 / 46.5 -> 45.0 at 32,768 (64 tokens), 71.6 -> 72.1 / 72.8 -> 70.4 / 73.2 -> 71.9 at 65,536.
// Forks of one prefix read the same bytes, so what one of them left in the cache is there for the next: their calls do so only where the
// keys are more than it holds (eight forks of 32,768 tokens queried in turn, 32 tokens each, 33.1 -> 36.8 us a query from 88 MiB on).
constexpr int64_t kStreamMinBytes = int64_t(88) << 20, kLastLevelBytes = int64_t(256) << 20;
bool streams_once(const sk_pool* p, int64_t cached, int64_t longest, bool shared)
{
    if (p->stream_min_tokens >= 0) return longest >= p->stream_min_tokens;
    return cached * p->d.n_kv_heads * p->d.head_dim * 2 * p->L.elem >= (shared ? kLastLevelBytes : kStreamMinBytes);
}

struct TileReq {            // one tile of query rows and the keys it may see
    int32_t tbl_off, q_tok0, n_tok;
    int32_t pos0;           // absolute position of its first token, or SK_NO_CAUSAL
    int32_t kv_vis;         // cached tokens visible to the tile (positions 0 .. kv_vis-1)
    int32_t eph_blk[2], eph_cnt[2], eph_pos0[2];
    int32_t hole_lo, hole_hi;   // evicted cached tokens of the session
    int32_t tok_period, sub_blocks;   // > 0: the tile packs sequences of tok_period tokens (see sk_work)
    int32_t alone;              // no other tile of the call reads the session's keys
    int32_t shared;             // the session holds blocks that other sessions hold too: other items of the call may read them
};
struct ListGroup {          // tiles that share a kernel variant and the q/out/lse arrays
    Variant v = {SK_KV_SIMPLE, 16, 1};
    const void* q = nullptr; void* out = nullptr; float* lse = nullptr;
    std::vector<TileReq> tiles;
};

// Cuts T tokens (packed rows q_row0..) that share `base` into row tiles of the group's height.
void add_tiles(ListGroup& g, const TileReq& base, int32_t q_row0, int32_t T)
{
    for (int32_t t0 = 0; t0 < T; t0 += g.v.tok_per_tile) {
        TileReq r = base;
        r.q_tok0 = q_row0 + t0;
        r.n_tok = std::min(g.v.tok_per_tile, T - t0);
        r.alone = base.alone && !base.shared && T <= g.v.tok_per_tile;
        if (base.pos0 < SK_NO_CAUSAL) {
            r.pos0 = base.pos0 + t0;
            r.kv_vis = std::min<int64_t>(base.kv_vis, int64_t(r.pos0) + r.n_tok);
        }
        g.tiles.push_back(r);
    }
}

// Pieces of at most `chunk` keys that a tile is cut into (a tile that sees no cached key is one piece), and which eighth of
// a chunk a piece's length falls into.  Lengths and chunks stay below 2^30.
uint32_t list_parts(const TileReq& t, uint32_t chunk) { return t.kv_vis > 0 ? ((uint32_t)t.kv_vis + chunk - 1) / chunk : 1; }
uint32_t list_bucket(uint32_t len, uint32_t chunk) { return len == chunk ? 8 : uint32_t(uint64_t(len) * 8 / chunk); }

// Length of the pieces a launch's tiles are cut into: the one for which the launch is expected to end first.
// The workgroups are taken up in order by the CUs that become free (those of a KV head by that head's share of
// the CUs), so the end is that of a list schedule; more pieces end more evenly, but each costs its start and
// end and a partial that the combine kernel reads back.  Times in us, measured: an iteration of 64 keys in the
// 256-row kernel 1.7 (one workgroup per CU); in the smaller ones 1.4 with one workgroup per CU and 2.7 with
// two (the stream from HBM); start and end of a workgroup 6; a partial of 128 rows 0.018 (with the present start, end and combine launch,
// 31 random steps that they decide: ends of 4 choose 0.3 % slower pieces, of 7 0.4 % faster ones, 0.012 3.5 % slower ones).
// Measured against pieces of one length for about 2,048 workgroups, in session order: 48-session step 4.58 ->
// 4.05 ms (append launch 4.25 -> 3.76: no 19,648-key pieces that end in a ragged last round, tiles whole and
// longest first; combine kernels 0.16 -> 0.02); 64 questions at 64K 1.13 -> 1.04 ms (7 pieces per tile, 3.5
// rounds of the chip -> 2 pieces, one round).
// The schedule is only played through where simple bounds of its end (the average load, the longest piece) do not
// say already that the length is no better, and no further than to where it is known to be none.
// head_dim 64 on the matrix pipe has times of its own (ListCost), with the uncommitted tokens of a tile.  0 is returned where no length
// is expected to end before `bound`.  Fitted to 13,000 timed launches of 992 steps and question batches.
// `step`: what lists beyond 16 KiB count, with `other_bytes` beside this launch's.  The length of the pieces is chosen with nothing, as
// the scatter launch carries such lists (launch_list) for less than the times err: with the 14 us of the copy that they once needed,
// plans stayed under 16 KiB (of 850 random steps and 650 question batches 146 and 234 are cut otherwise, at 0.85 and 0.93 of their time in
// the geometric mean, six steps and three batches more than 3 % slower, up to 8).
struct ListCost {
    double start, it_alone, it_shared, ends;     // as in RegCost
    double segment;                              // start of a run of uncommitted tokens
};
constexpr ListCost kList256d64 = {2.0, 0.88, 0.16, 6.4, 1.05}, kList128d64 = {1.8, 0.87, 0.29, 5.2, 0.75}, kList64d64 = {3.8, 0.63, 0.0, 2.6, 0.75};
constexpr size_t kUploadStep = 16384;        // bytes of lists beyond which a copy of them takes 14 us longer (launch_list)
bool list_narrow(const sk_pool* p, const Variant& v) { return p->d.head_dim == 64 && p->L.elem == 2 && v.id != SK_KV_SIMPLE; }

int64_t list_chunk(const sk_pool* p, const ListGroup& g, double step = 0.0, size_t other_bytes = 0, double* expected_us = nullptr,
                   size_t* expected_bytes = nullptr, double bound = HUGE_VAL)
{
    int64_t longest = 0;
    for (const TileReq& t : g.tiles) longest = std::max<int64_t>(longest, t.kv_vis);
    const int Hkv = p->d.n_kv_heads;
    const bool big = g.v.id == SK_KV_MFMA256, narrow = list_narrow(p, g.v);
    const ListCost& nc = big ? kList256d64 : g.v.id == SK_KV_MFMA128 ? kList128d64 : kList64d64;
    const size_t n_tiles = g.tiles.size();
    if (n_tiles == 0 || (longest == 0 && !narrow)) return 256;
    double best = 0; int64_t best_chunk = 0, last = 0;
    std::vector<double> lane;                              // when each lane is free: a heap, the first one on top
    std::vector<int32_t> rest(n_tiles);                    // iterations of each tile's last piece
    std::vector<double> ordered(n_tiles);                  // how long that piece takes, longest eighths first
    std::vector<uint8_t> bucket(n_tiles), own_its(n_tiles), own_runs(n_tiles);
    for (size_t i = 0; narrow && i < n_tiles; ++i) {
        const TileReq& t = g.tiles[i];
        const int32_t subs = t.tok_period > 0 ? (t.n_tok + t.tok_period - 1) / t.tok_period : 1;
        int32_t its = 0, runs = 0;
        for (int e = 0; e < 2; ++e)
            if (t.eph_cnt[e] > 0) { const int32_t n = e == 1 ? subs : 1; its += n * ((t.eph_cnt[e] + 63) / 64); runs += n; }
        own_its[i] = (uint8_t)std::min(its, 255); own_runs[i] = (uint8_t)std::min(runs, 255);
    }
    for (int64_t k = 1; k <= 256; k += std::max<int64_t>(1, k / 4)) {
        const int64_t chunk = std::max<int64_t>(256, ((longest + k - 1) / k + 63) / 64 * 64);
        if (chunk == last) { if (chunk == 256) break; continue; }
        last = chunk;
        int64_t whole = 0, parts = 0, split = 0, its_sum = 0, its_max = 0, runs = 0;
        size_t count[9] = {};
        for (size_t i = 0; i < n_tiles; ++i) {
            const uint32_t np = list_parts(g.tiles[i], (uint32_t)chunk), left = (uint32_t)g.tiles[i].kv_vis - (np - 1) * (uint32_t)chunk;
            if (np > 1) { parts += np; ++split; }
            whole += np - 1;
            rest[i] = int32_t((left + 63) / 64) + own_its[i];
            runs += own_runs[i];
            bucket[i] = (uint8_t)list_bucket(left, (uint32_t)chunk);
            ++count[bucket[i]];
            its_sum += rest[i]; its_max = std::max<int64_t>(its_max, rest[i]);
        }
        const int64_t n = whole + (int64_t)n_tiles;
        const bool sparse = big || (!narrow && n * Hkv <= p->n_cus);
        const double room = double(p->n_cus) * (big ? 1 : 2);
        const double it = narrow ? nc.it_alone + nc.it_shared * std::min(1.0, double(n * Hkv) / room) : big ? 1.7 : sparse ? 1.4 : 2.7;
        const double ends = narrow ? nc.ends : 6.0, segment = narrow ? nc.segment : 0.0;
        const int64_t lanes = std::max<int64_t>(1, int64_t(p->n_cus) * (sparse ? 1 : 2) / Hkv);
        const size_t bytes = (size_t)(n * Hkv) * sizeof(sk_work) + (size_t)(split * Hkv) * sizeof(sk_comb);
        const double carried = narrow && other_bytes + bytes > kUploadStep ? step : 0.0;
        const double merge = carried + (!narrow ? double(parts) * Hkv * 0.018 * g.v.rows_per_slot / 128.0
                                     : split == 0 ? 0.0 : 4.0 + double(Hkv * g.v.rows_per_slot) * 1e-3 * (0.018 * double(parts) + 0.19 * double(split)));
        // whole chunks fill the lanes evenly; the rest goes to whichever lane is free first
        const double c = double(chunk / 64) * it + ends, base = c * double(whole / lanes);
        const int64_t ahead = whole % lanes;               // lanes with one whole chunk more than the others
        auto no_better = [&](double end) { return !(end + merge < (best_chunk != 0 ? 0.995 * best : bound)); };
        double end = std::max(ahead > 0 ? base + c : base, base + (double(its_max) * it + ends));
        const double load = (double(whole) * c + double(its_sum) * it + double(n_tiles) * ends + double(runs) * segment) / double(lanes);
        if (narrow && no_better(load * (1 - 1e-9))) break;      // (neither the load nor the rest gets less with shorter pieces)
        if (no_better(std::max(end, load * (1 - 1e-9)))) continue;
        if ((int64_t)n_tiles > lanes - ahead) {            // (else each gets a lane that is free at `base`)
            size_t at[9], sum = 0;
            for (int b = 8; b >= 0; --b) { at[b] = sum; sum += count[b]; }
            for (size_t i = 0; i < n_tiles; ++i) ordered[at[bucket[i]]++] = double(rest[i]) * it + double(own_runs[i]) * segment + ends;
            lane.assign((size_t)lanes, base + c);
            std::fill(lane.begin(), lane.begin() + (lanes - ahead), base);
            for (size_t i = 0; i < n_tiles && !no_better(end); ++i) {
                const double x = lane[0] + ordered[i];
                end = std::max(end, x);
                size_t hole = 0;                           // x takes its place in the heap from the top
                for (size_t kid = 1; kid < (size_t)lanes; kid = 2 * hole + 1) {
                    if (kid + 1 < (size_t)lanes && lane[kid + 1] < lane[kid]) ++kid;
                    if (!(lane[kid] < x)) break;
                    lane[hole] = lane[kid]; hole = kid;
                }
                lane[hole] = x;
            }
            if (no_better(end)) continue;
        }
        for (size_t i = 0; narrow && (int64_t)n_tiles <= lanes - ahead && i < n_tiles; ++i) end = std::max(end, base + (double(rest[i]) * it + double(own_runs[i]) * segment + ends));
        if (no_better(end)) continue;
        best = end + merge; best_chunk = chunk;
        if (expected_us) *expected_us = end + merge - carried + nc.start + 2.0;       // (with the launch itself)
        if (expected_bytes) *expected_bytes = bytes;
    }
    return best_chunk;
}

// Expected time of a call's launches (head_dim 64), or something not below `bound`; `step` as in list_chunk, counted once.
double list_cost(const sk_pool* p, const ListGroup* const* groups, int n_groups, size_t scatter_bytes, double step, double bound = HUGE_VAL)
{
    double us = 0;
    size_t least = scatter_bytes, bytes = scatter_bytes;
    for (int gi = 0; gi < n_groups; ++gi) least += groups[gi]->tiles.size() * p->d.n_kv_heads * sizeof(sk_work);
    for (int gi = 0; gi < n_groups; ++gi) {
        const ListGroup& g = *groups[gi];
        if (g.tiles.empty()) continue;
        double end = 0;
        size_t b = 0;
        if (list_chunk(p, g, step, least - g.tiles.size() * p->d.n_kv_heads * sizeof(sk_work), &end, &b, bound - us) == 0) return bound;
        us += end; bytes += b;
    }
    return us + (bytes > kUploadStep ? step : 0.0);
}

// Expected time, in us, of the attention and combine launches of a single-session call whose row tiles are cut into pieces of
// `chunk` keys, with `own` uncommitted tokens as one more piece of each tile.  The workgroups are played through in the order the
// hardware takes them: workgroup b goes to XCD b % 8, where its shader engine is the next of four in turn, and waits there until
// one of the engine's CUs is free, with all behind it on that XCD waiting too.  So an even share per CU is not enough: the
// workgroups of splits that a tile does not have end at once but take their turn, and an engine that got more of the long pieces
// holds up the others (700 tokens of 12/4 heads behind 2,600: 47 us in pieces of 384 keys, 35 in pieces of 576; a schedule over any free CU
// expects 32 and 33).  Fitted to 39,000 timed launches of 3,330 calls (0 to 131,072 cached tokens, 9 to 3,300 new ones, 13 layer shapes).
// Returns early with something not below `stop` where the end cannot be below it; *all_above: shorter pieces will not be either (their
// load and merge are no less).
struct RegCost {
    double start;                    // of the launch, against that of the other instances of the head_dim
    double it_alone, it_shared;      // an iteration of 64 keys with the chip empty, and what is added when all of it is busy
    double ends;                     // start and end of a workgroup
    double merge, part, row;         // combine launch; 1,000 rows of a partial written and read; 1,000 rows merged
};
// (Start, end and combine launch have become about 1 us shorter each since: tried again on 83 random appends of 128 dims and 214 of 64 that
// they decide, ends of 6 and 7, merge of 0.3, row of 0.3 and part of 0.04 choose 0.0 to 0.4 % slower pieces, and the first rule 8 to 11 %;
// the best piece among those of seven such settings is 1.4 to 1.7 % faster than the chosen one.)
constexpr RegCost kCost256 = {0.0, 1.1, 0.47, 8.0, 1.0, 0.05, 0.45}, kCost256d64 = {0.7, 0.9, 0.15, 2.7, 1.2, 0.08, 0.36},
                  kCost128d64 = {0.0, 0.9, 0.25, 2.2, 1.3, 0.08, 0.34};
double regular_end(const sk_pool* p, const Variant& v, int64_t n_tok, int32_t pos0, int64_t kv_len, int32_t own, int64_t chunk, double stop, bool* all_above)
{
    constexpr int kXcds = 8, kEngines = 4, kMaxLanes = 64;
    const bool big = v.id == SK_KV_MFMA256;
    const RegCost& c = p->d.head_dim == 128 ? kCost256 : big ? kCost256d64 : kCost128d64;
    const int Hkv = p->d.n_kv_heads, per_cu = big ? 1 : 2;
    const int64_t tiles = (n_tok + v.tok_per_tile - 1) / v.tok_per_tile, chunk_its = chunk / 64, own_its = (own + 63) / 64;
    auto visible = [&](int64_t tile) { return pos0 < SK_NO_CAUSAL ? std::min(kv_len, pos0 + std::min(n_tok, (tile + 1) * v.tok_per_tile)) : kv_len; };
    int64_t pieces = 0, parts = 0, split = 0, its = 0;
    for (int64_t t = 0; t < tiles; ++t) {
        const uint32_t kv = (uint32_t)visible(t), np = (kv + (uint32_t)chunk - 1) / (uint32_t)chunk + (own > 0 ? 1 : 0);
        pieces += np; its += (kv + 63) / 64 + own_its;
        if (np > 1) { parts += np; ++split; }
    }
    const double room = double(p->n_cus * per_cu), it = c.it_alone + c.it_shared * std::min(1.0, double(pieces * Hkv) / room);
    const double stage = own > 0 && (tiles > 1 || own > SK_STAGE_TOKENS) ? 2.5 : 0.0;      // a launch in front writes the own tokens to the staging area
    const double apart = c.start + stage + (split == 0 ? 0.0 : c.merge + double(Hkv * v.rows_per_slot) * 1e-3 * (c.part * double(parts) + c.row * double(split)));
    const double load = (double(its) * it + double(pieces) * c.ends) * Hkv / room;
    *all_above = apart + load >= stop;
    if (*all_above) return apart + load;
    const int64_t total = ((kv_len + chunk - 1) / chunk + (own > 0 ? 1 : 0)) * tiles * Hkv;
    if (double(total) <= room)                                 // nobody waits
        return apart + c.ends + it * double(std::max(std::min(chunk_its, (kv_len + 63) / 64), own_its));
    if (double(total) > 64.0 * room)                           // the end of so long a launch is a small part of it
        return apart + load + 0.5 * (c.ends + it * double(std::min(chunk_its, (kv_len + 63) / 64)));
    const int lanes = std::min(kMaxLanes, std::max(1, p->n_cus * per_cu / (kXcds * kEngines)));
    int stride = kXcds;                                        // XCDs that many apart get the same lengths
    for (int h = Hkv; h != 0;) { const int r = stride % h; stride = h; h = r; }
    double end = 0;
    for (int x = 0; x < kXcds; x += stride) {
        double free_at[kEngines][kMaxLanes];                   // heaps: the first CU to be free on top
        for (int e = 0; e < kEngines; ++e) std::fill(free_at[e], free_at[e] + lanes, 0.0);
        double turn = 0;
        int engine = 0;
        for (uint32_t b = (uint32_t)x; b < total; b += kXcds, engine = (engine + 1) % kEngines) {
            const uint32_t rest = b / (uint32_t)Hkv, part = rest / (uint32_t)tiles;
            const int64_t kv = visible(tiles - 1 - (rest - part * (uint32_t)tiles)), begin = part * chunk;
            double* heap = free_at[engine];
            turn = std::max(turn, heap[0]);
            double t = turn + 0.3;                             // a split the tile does not have
            const bool cached = begin < kv, last = own > 0 && !cached && begin - chunk < kv;
            if (cached || last) {
                t = turn + c.ends + it * double(last ? own_its : std::min(chunk_its, (kv - begin + 63) / 64));
                end = std::max(end, t);
                if (end + apart >= stop) return end + apart;
            }
            int hole = 0;                                      // t takes its place in the heap from the top
            for (int kid = 1; kid < lanes; kid = 2 * hole + 1) {
                if (kid + 1 < lanes && heap[kid + 1] < heap[kid]) ++kid;
                if (!(heap[kid] < t)) break;
                heap[hole] = heap[kid]; hole = kid;
            }
            heap[hole] = t;
        }
    }
    return end + apart;
}

// Length of the pieces for which that time is least, if it is below `best`.
int64_t regular_chunk(const sk_pool* p, const Variant& v, int64_t n_tok, int32_t pos0, int64_t kv_len, int32_t own, double& best)
{
    int64_t chosen = 0, last = 0;
    for (int64_t k = 1; k <= 256; k += k < 64 ? 1 : k / 4) {
        const int64_t chunk = std::max<int64_t>(256, ((kv_len + k - 1) / k + 63) / 64 * 64);
        if (chunk == last) { if (chunk == 256) break; continue; }
        last = chunk;
        bool all_above = false;
        const double stop = chosen ? 0.995 * best : best, end = regular_end(p, v, n_tok, pos0, kv_len, own, chunk, stop, &all_above);
        if (all_above) break;
        if (end < stop) { best = end; chosen = chunk; }
    }
    return chosen;
}

int plan_regular(const sk_pool* p, int32_t id, int64_t n_tok, int32_t pos0, int64_t kv_len, int32_t eph_cnt, int32_t eph_pos0,
                 int64_t hole_lo, int64_t hole_hi, int32_t n_splits_req, RegPlan& R)
{
    Variant& v = R.v;
    if (!pick_variant(p, n_tok, v, !p->no_256, kv_len)) return SK_E_SHAPE;
    sk_launch& L = R.L;
    memset(&L, 0, sizeof L);
    L.rows_per_slot = v.rows_per_slot;
    L.mode = SK_MODE_REGULAR;
    L.tbl_off = int32_t(int64_t(id) * p->L.max_blocks_per_session);
    L.n_tok = (int32_t)n_tok;
    L.tok_per_tile = v.tok_per_tile;
    L.n_tiles = int32_t((n_tok + v.tok_per_tile - 1) / v.tok_per_tile);
    L.pos0 = pos0;
    L.kv_len = (int32_t)kv_len;
    L.hole_lo = (int32_t)hole_lo; L.hole_hi = (int32_t)hole_hi;
    L.by_heads = sk_make_div((uint32_t)p->d.n_kv_heads);
    if (v.id == SK_KV_SMALL) return plan_small(p, kv_len, eph_cnt, n_splits_req, R);
    if (p->L.elem == 4) return plan_f32(p, kv_len, eph_cnt, n_splits_req, R);
    int64_t base_wgs = int64_t(L.n_tiles) * p->d.n_kv_heads;
    const int64_t slots_rows = p->L.part_slots * kPartSlotRows;
    const int has_eph = eph_cnt > 0 ? 1 : 0;
    int64_t S;
    if (n_splits_req > 0) S = n_splits_req;
    else {
        // A call with few row tiles (a query) is bound by streaming the cache once: one workgroup
        // per CU measured faster than two (fewer split partials to write and merge).  Calls with
        // many row tiles (appends) are bound by arithmetic and want two workgroups per CU.
        // Not so with head_dim 64, whose smaller workgroups overlap on a CU (us per query, one -> two per CU, 32/8 heads):
        //   128 rows   14,800 cached 16.9 -> 16.4, 32,768 25.1 -> 22.0, 65,536 41.5 -> 38.6, 131,072 73.9 -> 62.5
        //    64 rows   14,800 14.3 -> 14.7, 20,000 15.9 -> 16.2, 26,000 18.4 -> 17.9, 32,768 20.9 -> 20.0, 65,536 33.3 -> 29.3, 131,072 59.3 -> 49.1
        // (three: 25.0 at 32,768 with 128 rows, 52.7 at 131,072 with 64)
        const bool two_per_cu = p->d.head_dim == 64 && (v.id == SK_KV_MFMA128 || (v.id == SK_KV_MFMA64 && kv_len >= 24576));
        const int64_t target = p->target_wgs_set ? p->target_wgs : (((L.n_tiles <= 2 && !two_per_cu) || v.id == SK_KV_MFMA256) ? 256 : 512);
        S = std::max<int64_t>(1, (target + base_wgs / 2) / base_wgs);
    }
    int64_t chunk = kv_len > 0 ? (kv_len + S - 1) / S : 64;
    // The 256-row instance: by the expected end of the launches (regular_end).  One workgroup to a CU makes the number of
    // workgroups count: with the pieces cut for about 256 of them, 264 were two rounds of the chip.
    // us per append, pieces for about 256 workgroups -> by a schedule of longest pieces first over any free CU -> by the order of the launch:
    //   32/8 d 128    1,500 tokens behind 1 cached 53.6 -> 58.3 -> 51.4, 1,750 behind 1 60.0 -> 68.6 -> 57.6, 1,500 behind 600 65.4 -> 76.7 -> 63.3,
    //                 1,200 into an empty session 55.5 -> 39.8 -> 39.7, 700 behind 32,512 521 -> 351 -> 353
    //   28/4 d 128    2,000 behind 1 63.0 -> 68.3 -> 60.7;  12/4 d 128  700 behind 2,600 37.4 -> 43.6 -> 34.0;  16/16 d 128  1,200 at 0 41.1 -> 43.1 -> 33.0
    //   14/2 d 64     2,000 at 0 53.8 -> 43.7 -> 36.1;  32/8 d 64  2,000 behind 1 52.9 -> 58.1 -> 47.7
    // Over 770 appends (0 to 32,512 cached, 200 to 3,376 tokens, seven layer shapes), against the first rule: 0.89 (128 dims) and 0.80 (64) of its time in the
    // geometric mean, one of them more than 3 % slower (3.8); with the second 0.91 and 0.83, and 63 of them more than 3 % slower, up to 17.
    if (n_splits_req <= 0 && !p->target_wgs_set && v.id == SK_KV_MFMA256 && kv_len > 0) {
        double best = HUGE_VAL;
        chunk = regular_chunk(p, v, n_tok, pos0, kv_len, eph_cnt, best);
        if (p->d.head_dim == 64) {
            // 128-row tiles of four waves, two workgroups to a CU, where they are expected to end earlier: less padding, or an evener
            // end
            const Variant low = {SK_KV_MFMA128, 128, 128 / p->L.G};
            const int64_t chunk128 = regular_chunk(p, low, n_tok, pos0, kv_len, eph_cnt, best);
            if (chunk128 > 0) {
                v = low; chunk = chunk128;
                L.rows_per_slot = v.rows_per_slot; L.tok_per_tile = v.tok_per_tile;
                L.n_tiles = int32_t((n_tok + v.tok_per_tile - 1) / v.tok_per_tile);
                base_wgs = int64_t(L.n_tiles) * p->d.n_kv_heads;
            }
        }
    }
    // at least four 64-key iterations per workgroup of the matrix-pipe kernels; the fp32-FMA kernel
    // (32-key tiles, far slower per key) takes shorter pieces so that small caches still spread over the chip
    if (n_splits_req <= 0) chunk = std::max<int64_t>(chunk, v.id == SK_KV_SIMPLE ? 64 : 256);
    chunk = (chunk + 63) / 64 * 64;
    S = kv_len > 0 ? (kv_len + chunk - 1) / chunk : 0;
    int64_t parts = std::max<int64_t>(1, S + has_eph);
    // respect the partial-slot capacity
    while (parts > 1 && base_wgs * parts * v.rows_per_slot > slots_rows) {
        chunk *= 2;
        S = kv_len > 0 ? (kv_len + chunk - 1) / chunk : 0;
        parts = std::max<int64_t>(1, S + has_eph);
        if (S <= 1) break;
    }
    if (parts > 1 && base_wgs * parts * v.rows_per_slot > slots_rows) return SK_E_WORKSPACE;
    if (base_wgs * parts > (int64_t(1) << 30)) return SK_E_WORKSPACE;
    L.chunk = (int32_t)chunk;
    L.n_splits = (int32_t)parts;
    L.by_tiles = sk_make_div((uint32_t)L.n_tiles); L.by_chunk = sk_make_div((uint32_t)chunk);
    L.eph_blk[0] = 0; L.eph_cnt[0] = eph_cnt; L.eph_pos0[0] = eph_pos0;
    // Small queries (at most 64 rows per KV head; every cached token visible to every row): the splits
    // interleave their 64-key pieces.  Measured 3-5 % faster there (16 tokens at 128K: 99.5 -> 96 us),
    // 2-3 % slower for the 128-row instance, which keeps contiguous chunks.  Larger blocks gain more
    // (16 tokens at 128K: 98 / 96 / 92 us with 16- / 64- / 256-token blocks).
    L.interleave = (!p->no_interleave && v.id == SK_KV_MFMA64 && S > 1 && kv_len <= (int64_t)pos0) ? 1 : 0;
    L.by_step = sk_make_div((uint32_t)(S * 64));
    R.base_wgs = (int32_t)base_wgs; R.parts = (int32_t)parts; R.wgs = int32_t(base_wgs * parts); R.kv_len = kv_len;
    // On request (SK_FUSE=1) the ring kernels merge their split partials themselves (one launch per
    // call).  Workgroups only wait for each other when the whole launch fits on the device at once (the
    // 256-row instance holds a CU alone, the others share it in pairs); otherwise the last workgroup of a
    // unit merges alone.  Not the default: a device-scope round trip (atomic, coherent load) measured about
    // 3 us on this hardware and the scheme needs four in a row, against 4-7 us for the combine kernel.
    const bool mfma = v.id != SK_KV_SIMPLE;
    // A 128-row call that gives every CU at most one workgroup takes the eight-wave instance: two key
    // phases per row group, so a wave has half the arithmetic per 64 keys and its SIMD a second wave
    // to overlap it with.  They pay off once what a workgroup streams outweighs their longer start and their merge of the two phases.
    // Measured (us per query, four waves -> eight, by the keys of a workgroup, 256 workgroups; three sessions in turn):
    //   heads, rows    256               384               448               512               1,024
    //    8/1, 128      24.7 -> 25.3      27.6 -> 27.5      29.1 -> 28.8      30.2 -> 30.0      -
    //   14/2, 126      20.0 -> 20.7      23.0 -> 23.0      24.5 -> 24.2      25.7 -> 25.3      38.8 -> 38.4
    //   28/4, 126      17.9 -> 18.5      20.9 -> 20.9      22.1 -> 21.9      23.4 -> 22.9      36.9 -> 35.9
    //   32/8, 128      17.7 -> 18.3      20.6 -> 20.6      21.9 -> 21.7      23.2 -> 22.7      36.1 -> 35.1
    //   64/16, 128     17.4 -> 18.0      20.1 -> 20.3      21.6 -> 21.4      22.9 -> 22.5      35.2 -> 34.4
    //   32/32, 128     17.6 -> 18.2      20.5 -> 20.5      21.8 -> 21.6      23.1 -> 22.7      35.4 -> 34.5
    // (break-even lies at 384 to 448 keys since the phases' merge got shorter; what 448 would gain on 512 is 1 %)
    const bool long_enough = p->p128_min_tokens >= 0 ? kv_len >= p->p128_min_tokens : chunk >= kP128MinKeys;
    if (p->p128 && v.id == SK_KV_MFMA128 && p->d.head_dim == 128 && R.wgs <= p->n_cus && long_enough) v.id = SK_KV_MFMA128P;
    L.fuse = (p->fuse && mfma && parts > 1 && base_wgs <= p->L.sync_units && parts < 65536) ? 1 : 0;
    const int64_t resident = int64_t(p->n_cus) * ((v.id == SK_KV_MFMA256 || v.id == SK_KV_MFMA128P) ? 1 : 2);
    L.wait_polls = (L.fuse && R.wgs <= resident) ? p->wait_polls : 0;
    L.merge_fences = p->merge_fences ? 1 : 0;
    // With one row tile per KV head no two workgroups read the same keys, and the kernel can load them non-temporal: the 64-row
    // instance always does, the 128-row ones by streams_once, the 256-row one (and every call whose row tiles share their keys
    // through the L2) never.
    const bool once_pays = v.id == SK_KV_MFMA64 || ((v.id == SK_KV_MFMA128 || v.id == SK_KV_MFMA128P) && streams_once(p, kv_len, kv_len, holds_shared(p, p->sessions[id])));
    L.kv_once = (!p->no_stream_loads && L.n_tiles == 1 && once_pays) ? 1 : 0;
    return SK_OK;
}

// Enqueues a planned call.
int launch_regular(sk_pool* p, RegPlan& R, const void* q, void* out, int out_dtype, float* lse, hipStream_t st)
{
    if (inject(p, SK_SITE_ATTENTION)) return SK_E_HIP;
    if (!p->device) return SK_OK;
    sk_launch L;
    fill_launch_common(p, L, q, out, out_dtype, lse, R.v);
    {   // the plan holds everything but the pointers
        sk_launch& S = R.L;
        S.g = L.g; S.q = L.q; S.out = L.out; S.lse = L.lse; S.part_ml = L.part_ml; S.part_o = L.part_o; S.sync = L.sync;
        S.out_dtype = L.out_dtype; S.own_k = R.own_k; S.own_v = R.own_v;
    }
    const int32_t pc = prof_call(p);
    void *e0, *e1;
    prof_pair(p, pc, 0, &e0, &e1);
    int e;
    if (R.L.own_mode != SK_OWN_NONE) {
        R.commit.first_wg = R.commit_items > 0 ? R.wgs : INT32_MAX;
        R.commit.tables_rw = (int32_t*)((unsigned char*)p->d.workspace + p->L.off_tables);
        R.commit.kv_rw = (unsigned char*)p->d.kv_mem;
        e = sk_launch_attention_small(R.L, R.commit, R.wgs + R.commit_items * p->d.n_kv_heads, st, e0, e1);
    } else e = sk_launch_attention(R.L, R.v.id, R.wgs, st, e0, e1);
    if (e) { g_last_hip = e; return SK_E_HIP; }
    p->stats.launches++;
    R.enqueued = true;
    if (R.parts > 1 && !R.L.fuse) {
        // the attention kernel is enqueued and will write its partials; a failure here leaves out/lse unwritten
        prof_pair(p, pc, 1, &e0, &e1);
        e = inject(p, SK_SITE_COMBINE) ? (int)hipErrorUnknown : sk_launch_combine(R.L, R.base_wgs, R.parts, p->d.n_kv_heads, st, e0, e1);
        if (e) { g_last_hip = e; return SK_E_HIP; }
        p->stats.launches++;
    }
    p->stats.kv_bytes_streamed += R.kv_len * 2 * p->d.n_kv_heads * p->d.head_dim * p->L.elem * R.L.n_tiles;
    p->last.workgroups = R.wgs; p->last.n_splits = R.parts; p->last.row_tiles = R.L.n_tiles; p->last.kernel_variant = R.v.id;
    p->last.fused_merge = R.L.fuse;
    return SK_OK;
}

// Builds the scatter list for `count` tokens (packed rows src0..) going either behind position
// `dst_tok0` of session `s` (blocks already in s->blocks) or into staging blocks eph_blk0..
int build_scatter(const sk_pool* p, const Session* s, int32_t id, int64_t dst_tok0, int32_t src0, int64_t count,
                  int64_t first_new_block, bool to_eph, int64_t eph_blk0, std::vector<sk_scatter>& out)
{
    const int64_t B = to_eph ? 16 : p->d.block_tokens;
    for (int64_t t = dst_tok0; t < dst_tok0 + count;) {
        const int64_t gend = std::min<int64_t>((t / 16 + 1) * 16, dst_tok0 + count);
        sk_scatter it;
        const int64_t bi = t / B;
        it.src_tok0 = src0 + int32_t(t - dst_tok0);
        it.count = int32_t(gend - t);
        it.dst_slot0 = int32_t(t % B);
        it.to_eph = to_eph ? 1 : 0;
        if (to_eph) {
            it.dst_off = (eph_blk0 + bi) * p->L.eph_blk_stride;
            it.tbl_index = -1; it.block_id = 0;
        } else {
            const int32_t blk = s->blocks[bi];
            it.dst_off = int64_t(blk) * p->L.blk_stride;
            it.block_id = blk;
            it.tbl_index = (bi >= first_new_block) ? int32_t(int64_t(id) * p->L.max_blocks_per_session + bi) : -1;
        }
        out.push_back(it);
        t = gend;
    }
    return SK_OK;
}

// A single-session scatter in two halves, so that everything that can refuse the call happens before
// the call changes anything: scatter_reserve (size check, and a pinned ring slot if the list is too
// long to travel in the kernel arguments), then, once the list is built, scatter_launch.
struct ScatterSlot { bool upload = false; int slot = 0; unsigned char* host = nullptr; };

int64_t scatter_groups(int64_t dst_tok0, int64_t count)     // 16-token groups the tokens dst_tok0 .. +count-1 touch
{
    return count <= 0 ? 0 : (dst_tok0 + count + 15) / 16 - dst_tok0 / 16;
}

constexpr size_t kListInPlaceMax = 8192;     // groups up to which the commit kernel reads its list in the pinned slot (scatter_launch)

int scatter_reserve(sk_pool* p, int64_t n_items, ScatterSlot& ss)
{
    ss = ScatterSlot();
    if (n_items <= SK_SCATTER_ARGS_MAX) return SK_OK;
    if (size_t(n_items) * sizeof(sk_scatter) > p->L.meta_bytes) return SK_E_WORKSPACE;
    ss.upload = true;
    return ring_acquire(p, &ss.slot, &ss.host);
}

int scatter_launch(sk_pool* p, const ScatterSlot& ss, const std::vector<sk_scatter>& items, const void* k, const void* v, hipStream_t st)
{
    if (items.empty()) return SK_OK;
    unsigned char* ws = (unsigned char*)p->d.workspace;
    if (!ss.upload) {          // short list: in the kernel arguments, nothing to upload
        if (inject(p, SK_SITE_SCATTER)) return SK_E_HIP;
        if (!p->device) return SK_OK;
        sk_scatter_list lst;
        memcpy(lst.item, items.data(), items.size() * sizeof(sk_scatter));
        int e = sk_launch_scatter_args(p->geom, k, v, lst, (int32_t)items.size(), (int32_t*)(ws + p->L.off_tables),
                                       (unsigned char*)p->d.kv_mem, ws + p->L.off_eph, st);
        if (e) { g_last_hip = e; return SK_E_HIP; }
        p->stats.launches++;
        return SK_OK;
    }
    // A longer one is read where it lies, in the pinned slot: every KV head's workgroup of a group reads its 32 bytes over the host
    // link, one round trip where a copy in front is a launch of its own.  us per commit in a stream of them, and alone (a wait
    // behind each); copied -> read in place:
    //   heads       1,300 tokens             2,600                     10,400                  41,600                  131,072
    //   1  d 128    10.1 ->  7.4/23 -> 23    10.8 ->  8.5/23 -> 26     23 -> 10/30 -> 33       29 ->  18/ 44 ->  68    46 ->  43/ 78 ->  78
    //   2  d 64     10.3 ->  7.7/22 -> 26    10.7 ->  8.3/23 -> 26     23 -> 11/30 -> 31       29 ->  23/ 43 ->  74    48 ->  58/ 79 -> 103
    //   8  d 128    10.2 ->  7.8/23 -> 26    11.1 ->  9.0/24 -> 30     34 -> 19/40 -> 44       78 ->  63/ 94 ->  84   214 -> 194/252 -> 236
    //   32 d 128    13.2 -> 12.6/27 -> 31    19.4 -> 19.0/33 -> 40     82 -> 67/88 -> 81      276 -> 259/293 -> 285   -
    // With its attention behind it an append gains 1 to 3 us up to 4,096 tokens, alone as well (2,600 tokens of 32/8 heads into an
    // empty session and a question: 97.7 -> 96.2, alone 111.9 -> 110.9).  A commit that somebody waits for loses some; in a stream
    // only the longest of two heads of 64 dims does, which reads as much of the list for a quarter of the bytes.  Up to 8,192 groups,
    // as far as it was measured; longer lists are copied to the workspace.
    if (ss.host) memcpy(ss.host, items.data(), items.size() * sizeof(sk_scatter));
    const sk_scatter* list = (const sk_scatter*)ss.host;
    const bool in_place = items.size() <= kListInPlaceMax;
    if (!in_place) {
        int rc = ring_upload(p, ss.slot, items.size() * sizeof(sk_scatter), st);
        if (rc) return rc;
        list = (const sk_scatter*)(ws + p->L.off_meta);
    } else if (inject(p, SK_SITE_UPLOAD)) return SK_E_HIP;
    if (inject(p, SK_SITE_SCATTER)) return SK_E_HIP;
    if (!p->device) return SK_OK;
    int e = sk_launch_scatter(p->geom, k, v, list, (int32_t)items.size(),
                              (int32_t*)(ws + p->L.off_tables), (unsigned char*)p->d.kv_mem, ws + p->L.off_eph, st);
    if (in_place) ring_busy(p, ss.slot, st);         // whatever e is: an error that an earlier call left behind shows up here too, with the kernel on the stream
    if (e) { g_last_hip = e; return SK_E_HIP; }
    p->stats.launches++;
    return SK_OK;
}

bool overlap(const void* a, size_t na, const void* b, size_t nb)
{
    const uintptr_t x = reinterpret_cast<uintptr_t>(a), y = reinterpret_cast<uintptr_t>(b);
    return a && b && x < y + nb && y < x + na;
}

// Whether a call of T tokens writes its results over its own k or v.  Where the attention launch reads those in place, some of
// its workgroups would do so after others have written.
bool results_over_own(const sk_pool* p, int64_t T, const void* k, const void* v, const void* out, int out_dtype, const float* lse)
{
    const size_t kv = size_t(T) * p->d.n_kv_heads * p->d.head_dim * p->L.elem, rows = size_t(T) * p->d.n_q_heads;
    const size_t n_out = rows * p->d.head_dim * (out_dtype == SK_F32 ? 4 : 2);
    return overlap(out, n_out, k, kv) || overlap(out, n_out, v, kv) || overlap(lse, rows * 4, k, kv) || overlap(lse, rows * 4, v, kv);
}

// Copies a call's own k and v, as they are, to the staging area, which holds twice max_batch_tokens rows.
int copy_own(sk_pool* p, int64_t T, const void** k, const void** v, hipStream_t st)
{
    const size_t bytes = size_t(T) * p->d.n_kv_heads * p->d.head_dim * p->L.elem;
    unsigned char* to = (unsigned char*)p->d.workspace + p->L.off_eph;
    SK_HIP(hipMemcpyAsync(to, *k, bytes, hipMemcpyDeviceToDevice, st));
    SK_HIP(hipMemcpyAsync(to + bytes, *v, bytes, hipMemcpyDeviceToDevice, st));
    *k = to; *v = to + bytes;
    return SK_OK;
}

// Takes `need` blocks for the session (caller has checked availability).
void take_blocks(sk_pool* p, Session* s, int64_t need)
{
    for (int64_t i = 0; i < need; ++i) {
        s->blocks.push_back(p->free_blocks.front());
        p->refcnt[(size_t)p->free_blocks.front()] = 1;
        p->free_blocks.pop_front();
    }
    p->blocks_in_use += need;
}

// One session lets go of a block; the last holder returns it to the free list.
void release_block(sk_pool* p, int32_t b)
{
    if (--p->refcnt[(size_t)b] == 0) { p->free_blocks.push_back(b); p->blocks_in_use--; }
}

// After a fork, a truncation can leave the end of a session inside a block that other sessions
// also hold.  Before such a session appends it gets its own copy of that block: the one case of
// copy-on-write (nothing else ever writes into a block that is not the writer's alone).
bool tail_shared(const sk_pool* p, const Session* s)
{
    return s->len % p->d.block_tokens != 0 && p->refcnt[(size_t)s->blocks.back()] > 1;
}

// What an append changed in one session, so that a later failure of the same call can take it back.
struct Undo {
    Session* s = nullptr;
    int64_t len = 0;
    size_t n_blocks = 0;
    int32_t old_tail = -1;       // >= 0: the shared tail block that was swapped for a copy
};

// The caller has checked that a block is free.  The copy is ordered on `st` in front of the
// scatter that follows; the scatter also rewrites the table entry (it is told that the block is new).
// On failure nothing has changed.
int unshare_tail(sk_pool* p, Session* s, Undo& u, hipStream_t st)
{
    const int32_t old = s->blocks.back();
    const int32_t blk = p->free_blocks.front();
    if (inject(p, SK_SITE_BLOCK_COPY)) return SK_E_HIP;
    if (p->device) {
        int e = sk_launch_copy_block(p->geom, (unsigned char*)p->d.kv_mem, old, blk, st);
        if (e) { g_last_hip = e; return SK_E_HIP; }
    }
    p->free_blocks.pop_front();
    p->refcnt[(size_t)blk] = 1;
    p->refcnt[(size_t)old]--;                 // still held by the others
    p->blocks_in_use++;
    s->blocks.back() = blk;
    u.old_tail = old;
    return SK_OK;
}

// Takes an append back: the blocks it took return to the head of the free list in their old order,
// the length is restored; the copy of a shared tail is given up too unless `keep_copy` (the commit
// kernel is already enqueued and has pointed the device block table at the copy; keeping it changes
// nothing a caller can observe but the number of free blocks).
void rollback(sk_pool* p, const Undo& u, bool keep_copy)
{
    Session* s = u.s;
    while (s->blocks.size() > u.n_blocks) {
        const int32_t b = s->blocks.back();
        s->blocks.pop_back();
        p->refcnt[(size_t)b] = 0;
        p->free_blocks.push_front(b);
        p->blocks_in_use--;
    }
    if (u.old_tail >= 0 && !keep_copy) {
        const int32_t blk = s->blocks.back();
        s->blocks.back() = u.old_tail;
        p->refcnt[(size_t)u.old_tail]++;
        p->refcnt[(size_t)blk] = 0;
        p->free_blocks.push_front(blk);
        p->blocks_in_use--;
    }
    s->len = u.len;
}

// The host half of an append of T tokens to session s (availability already checked): copy of a
// shared tail, new blocks, new length.  Fills `u`; on failure nothing has changed.
int grow_session(sk_pool* p, Session* s, int64_t T, Undo& u, int64_t* first_new, hipStream_t st)
{
    u = Undo();
    u.s = s; u.len = s->len; u.n_blocks = s->blocks.size();
    const bool unshare = tail_shared(p, s);
    if (unshare) { int rc = unshare_tail(p, s, u, st); if (rc) return rc; }
    *first_new = (int64_t)s->blocks.size() - (unshare ? 1 : 0);
    take_blocks(p, s, blocks_needed(p, s->len, T));
    s->len += T;
    return SK_OK;
}

int check_out_dtype(const sk_pool* p, int out_dtype)
{
    if (out_dtype != SK_F32 && out_dtype != p->d.dtype) return SK_E_DTYPE;
    return SK_OK;
}

// ---- list mode: many row tiles (of several sessions, or of one question batch) in one launch ----

struct ScatterBatch { const void* k = nullptr; const void* v = nullptr; std::vector<sk_scatter> items; };

constexpr int kMaxGroups = 3;   // one launch per kernel variant in use

// A batched call in two halves.  plan_list cuts the tiles into workgroups, builds the lists and takes
// the pinned ring slot they travel in: everything that can refuse the call, and nothing that changes
// a session or the device.  launch_list uploads the lists and enqueues the kernels.
struct ListPlan {
    std::vector<sk_work> work[kMaxGroups];
    std::vector<sk_comb> comb[kMaxGroups];
    int64_t rows_base[kMaxGroups] = {};
    int64_t kv_total = 0, n_tiles = 0;
    bool fuse = false;
    int slot = 0;
    unsigned char* host = nullptr;
    bool scatter_enqueued = false;     // set by launch_list once a commit kernel is on the stream
};

int plan_list(sk_pool* p, const ScatterBatch* sb, int n_sb, ListGroup* groups, int n_groups, ListPlan& P)
{
    if (n_groups > kMaxGroups) return SK_E_INVAL;
    if (inject(p, SK_SITE_PLAN)) return SK_E_WORKSPACE;
    const int Hkv = p->d.n_kv_heads;
    P.kv_total = 0; P.n_tiles = 0;
    int64_t cached = 0, longest = 0;         // the call's keys that no two of its items read
    for (int gi = 0; gi < n_groups; ++gi)
        for (size_t i = 0; i < groups[gi].tiles.size(); ++i) {
            const TileReq& t = groups[gi].tiles[i];
            P.kv_total += t.kv_vis; ++P.n_tiles;
            if (!t.shared && (i + 1 == groups[gi].tiles.size() || groups[gi].tiles[i + 1].tbl_off != t.tbl_off)) cached += t.kv_vis;      // an item's last tile sees all of them
            longest = std::max<int64_t>(longest, t.kv_vis);
        }
    if (P.n_tiles == 0) return SK_OK;
    int64_t chunk_g[kMaxGroups];
    for (int gi = 0; gi < n_groups; ++gi) chunk_g[gi] = list_chunk(p, groups[gi]);
    const int64_t cap_rows = p->L.part_slots * kPartSlotRows;
    size_t bytes = 0;
    for (;;) {
        int64_t rows_used = 0;
        bool ok = true;
        int64_t unit = 0;
        for (int gi = 0; gi < n_groups && ok; ++gi) {
            ListGroup& g = groups[gi];
            const int64_t chunk = chunk_g[gi];
            P.work[gi].clear(); P.comb[gi].clear();
            P.rows_base[gi] = rows_used;
            int64_t slot = 0;       // in units of this group's rows_per_slot, from rows_base
            const bool once_pays = !p->no_stream_loads && (g.v.id == SK_KV_MFMA64 || (g.v.id == SK_KV_MFMA128 && streams_once(p, cached, longest, false)));
            struct Piece { int32_t tile, part, bucket; };
            std::vector<Piece> pieces, ordered;
            std::vector<int32_t> nparts(g.tiles.size()), slot0(g.tiles.size()), unit0(g.tiles.size());
            size_t n_pieces = 0, at[9] = {};
            for (size_t i = 0; i < g.tiles.size(); ++i) {
                const int32_t np = (int32_t)list_parts(g.tiles[i], (uint32_t)chunk);
                nparts[i] = np;
                n_pieces += (size_t)np;
                slot0[i] = np > 1 ? (int32_t)slot : -1;
                unit0[i] = np > 1 ? (int32_t)unit : -1;
                if (np > 1) { slot += int64_t(np) * Hkv; unit += Hkv; }
            }
            // In the order the workgroups start in: the longest pieces first (whole chunks, then what is left of
            // each tile, falling in eighths of a chunk), so that the launch ends evenly; among equals the tiles
            // of a session side by side, one part after the other, so that what runs at the same time reads
            // the same keys through the L2.
            pieces.reserve(n_pieces);
            size_t i0 = 0;
            while (i0 < g.tiles.size()) {
                size_t i1 = i0;
                int32_t max_parts = 1;
                for (; i1 < g.tiles.size() && g.tiles[i1].tbl_off == g.tiles[i0].tbl_off; ++i1) max_parts = std::max(max_parts, nparts[i1]);
                for (int32_t part = 0; part < max_parts; ++part)
                    for (size_t i = i0; i < i1; ++i)
                        if (part < nparts[i]) {
                            const int64_t len = std::min<int64_t>(g.tiles[i].kv_vis - int64_t(part) * chunk, chunk);
                            const int32_t bucket = (int32_t)list_bucket((uint32_t)len, (uint32_t)chunk);
                            pieces.push_back(Piece{(int32_t)i, part, bucket});
                            if (bucket > 0) ++at[bucket - 1];
                        }
                i0 = i1;
            }
            for (int b = 7; b > 0; --b) at[b - 1] += at[b];       // at[b]: pieces of longer eighths than b
            ordered.resize(n_pieces);
            for (const Piece& pc : pieces) ordered[at[pc.bucket]++] = pc;
            P.work[gi].reserve(n_pieces * (size_t)Hkv);
            for (const Piece& pc : ordered) {
                const TileReq& t = g.tiles[(size_t)pc.tile];
                const int32_t np = nparts[(size_t)pc.tile], part = pc.part, s0 = slot0[(size_t)pc.tile], u0 = unit0[(size_t)pc.tile];
                sk_work w = {};
                w.tbl_off = t.tbl_off; w.q_tok0 = t.q_tok0; w.n_tok = t.n_tok; w.pos0 = t.pos0;
                w.kv_begin = int32_t(part * chunk);
                w.kv_end = int32_t(std::min<int64_t>(t.kv_vis, (part + 1) * chunk));
                w.n_parts = np;
                w.hole_lo = t.hole_lo; w.hole_hi = t.hole_hi;
                w.tok_period = t.tok_period; w.sub_blocks = t.sub_blocks;
                w.once = t.alone && once_pays ? 1 : 0;
                if (part == np - 1)
                    for (int e = 0; e < 2; ++e) { w.eph_blk[e] = t.eph_blk[e]; w.eph_cnt[e] = t.eph_cnt[e]; w.eph_pos0[e] = t.eph_pos0[e]; }
                for (int h = 0; h < Hkv; ++h) {
                    w.kv_head = h;
                    w.part = np > 1 ? s0 + part * Hkv + h : -1;
                    w.unit = np > 1 ? u0 + h : -1;
                    w.part0 = np > 1 ? s0 + h : -1;
                    P.work[gi].push_back(w);
                }
            }
            for (size_t i = 0; i < g.tiles.size(); ++i) {
                if (nparts[i] < 2) continue;
                for (int h = 0; h < Hkv; ++h) {
                    sk_comb c = {};
                    c.part0 = slot0[i] + h; c.n_parts = nparts[i]; c.part_stride = Hkv;
                    c.q_tok0 = g.tiles[i].q_tok0; c.n_tok = g.tiles[i].n_tok; c.kv_head = h;
                    P.comb[gi].push_back(c);
                }
            }
            rows_used += slot * g.v.rows_per_slot;
            if (rows_used > cap_rows) ok = false;
        }
        // the last workgroup of a unit merges it inside the attention kernel when the call asks for
        // that (SK_FUSE_LIST) and every kernel in use can (the matrix-pipe instances)
        P.fuse = p->fuse_list && unit <= p->L.sync_units;
        for (int gi = 0; gi < n_groups; ++gi)
            if (!P.work[gi].empty() && groups[gi].v.id == SK_KV_SIMPLE) P.fuse = false;
        bytes = 0;
        for (int i = 0; i < n_sb; ++i) bytes += align_up(sb[i].items.size() * sizeof(sk_scatter), 256);
        for (int gi = 0; gi < n_groups; ++gi)
            bytes += align_up(P.work[gi].size() * sizeof(sk_work), 256) + align_up(P.comb[gi].size() * sizeof(sk_comb), 256);
        if (ok && bytes <= p->L.meta_bytes) break;
        if (chunk_g[0] > (int64_t(1) << 30)) return SK_E_WORKSPACE;
        for (int gi = 0; gi < n_groups; ++gi) chunk_g[gi] = std::min<int64_t>(2 * chunk_g[gi], int64_t(1) << 31);      // (longer than any session)
    }
    return ring_acquire(p, &P.slot, &P.host);
}

int launch_list(sk_pool* p, ListPlan& P, const ScatterBatch* sb, int n_sb, ListGroup* groups, int n_groups, int out_dtype, hipStream_t st)
{
    if (P.n_tiles == 0) return SK_OK;
    const int Hkv = p->d.n_kv_heads;
    // The lists, in the pinned slot as in the workspace: scatter lists, work lists, combine lists.  Up to 16 KiB one copy in front takes them there (2.5 us;
    // 16 beyond).  Beyond, the scatter lists are read where they lie, in the pinned slot, and items behind those of the first
    // copy the others (a launch of such items alone where there is nothing to scatter).  us per call, a copy in front -> by the
    // scatter launch: 3 sessions of 32/8 heads (24 KiB and more) 93.5 -> 77.0, 20 sessions 700 -> 685, 48 4,033 -> 4,009; 16 questions 92.7 ->
    // 80.8, of 64 dims 62.5 -> 50.3; below 16 KiB 4 questions 60.9 -> 62.6, of 64 dims 43.4 -> 45.0.  More groups than kListInPlaceMax
    // are copied too, as in scatter_launch.
    unsigned char* ws = (unsigned char*)p->d.workspace;
    unsigned char* dev_meta = p->device ? ws + p->L.off_meta : nullptr;
    size_t lists_bytes = 0, n_items = 0;
    int carrier = n_sb - 1;                     // the scatter list that carries the others
    for (int i = n_sb - 1; i >= 0; --i) { n_items += sb[i].items.size(); if (!sb[i].items.empty()) carrier = i; }
    for (int gi = 0; gi < n_groups; ++gi)
        lists_bytes += align_up(P.work[gi].size() * sizeof(sk_work), 256) + align_up(P.comb[gi].size() * sizeof(sk_comb), 256);
    const size_t stretch = size_t(Hkv) * 256, pieces = lists_bytes / 16, n_copies = (pieces + stretch - 1) / stretch;
    size_t off = 0, off_sb[2] = {0, 0}, off_work[kMaxGroups] = {}, off_comb[kMaxGroups] = {};
    bool in_place = lists_bytes + n_items * sizeof(sk_scatter) > kUploadStep && n_items <= kListInPlaceMax;
    auto place = [&]() {
        off = 0;
        for (int i = 0; i < n_sb; ++i) {
            off_sb[i] = off;
            off += align_up((sb[i].items.size() + (in_place && i == carrier ? n_copies : 0)) * sizeof(sk_scatter), 256);
        }
        for (int gi = 0; gi < n_groups; ++gi) {
            off_work[gi] = off; off += align_up(P.work[gi].size() * sizeof(sk_work), 256);
            off_comb[gi] = off; off += align_up(P.comb[gi].size() * sizeof(sk_comb), 256);
        }
    };
    place();
    if (off > p->L.meta_bytes) { in_place = false; place(); }          // (what plan_list has checked has no room for the copies' items)
    for (int i = 0; i < n_sb && P.host; ++i) {
        memcpy(P.host + off_sb[i], sb[i].items.data(), sb[i].items.size() * sizeof(sk_scatter));
        if (!in_place || i != carrier) continue;
        sk_scatter* more = (sk_scatter*)(P.host + off_sb[i]) + sb[i].items.size();
        for (size_t c = 0; c < n_copies; ++c) {
            sk_scatter it = {};
            it.to_eph = SK_COPY_LIST;
            it.src_tok0 = int32_t((off_work[0] - off_sb[i]) / 16 + c * stretch);
            it.count = int32_t(std::min(stretch, pieces - c * stretch));
            it.dst_off = int64_t(p->L.off_meta + off_work[0] + c * stretch * 16) - int64_t(p->L.off_eph);
            it.tbl_index = -1;
            more[c] = it;
        }
    }
    for (int gi = 0; gi < n_groups && P.host; ++gi) {
        memcpy(P.host + off_work[gi], P.work[gi].data(), P.work[gi].size() * sizeof(sk_work));
        memcpy(P.host + off_comb[gi], P.comb[gi].data(), P.comb[gi].size() * sizeof(sk_comb));
    }
    if (!in_place) { int rc = ring_upload(p, P.slot, off, st); if (rc) return rc; }
    else if (inject(p, SK_SITE_UPLOAD)) return SK_E_HIP;
    const unsigned char* scatter_lists = in_place ? P.host : dev_meta;
    for (int i = 0; i < n_sb; ++i) {
        const size_t n = sb[i].items.size() + (in_place && i == carrier ? n_copies : 0);
        if (n == 0) continue;
        if (!sb[i].items.empty() && inject(p, SK_SITE_SCATTER)) return SK_E_HIP;
        if (!p->device) continue;
        int e = sk_launch_scatter(p->geom, sb[i].k, sb[i].v, (const sk_scatter*)(scatter_lists + off_sb[i]), (int32_t)n,
                                  (int32_t*)(ws + p->L.off_tables), (unsigned char*)p->d.kv_mem, ws + p->L.off_eph, st);
        if (in_place) ring_busy(p, P.slot, st);            // whatever e is (see scatter_launch)
        if (e) { g_last_hip = e; return SK_E_HIP; }
        if (!sb[i].items.empty()) P.scatter_enqueued = true;
        p->stats.launches++;
    }
    if (inject(p, SK_SITE_ATTENTION)) return SK_E_HIP;
    if (!p->device) return SK_OK;
    const int32_t pc = prof_call(p);
    void *e0, *e1;
    sk_launch L[kMaxGroups];
    int32_t wgs = 0, max_parts = 1, most[kMaxGroups] = {};
    for (int gi = 0; gi < n_groups; ++gi) {
        if (P.work[gi].empty()) continue;
        ListGroup& g = groups[gi];
        fill_launch_common(p, L[gi], g.q, g.out, out_dtype, g.lse, g.v);
        L[gi].mode = SK_MODE_LIST;
        L[gi].part_ml += P.rows_base[gi] * 4;
        L[gi].part_o += P.rows_base[gi] * p->d.head_dim;
        L[gi].work = (const sk_work*)(dev_meta + off_work[gi]);
        L[gi].comb = (const sk_comb*)(dev_meta + off_comb[gi]);
        L[gi].fuse = P.fuse ? 1 : 0;
        L[gi].wait_polls = 0;          // the workgroups of a long list are not resident together
        L[gi].merge_fences = p->merge_fences ? 1 : 0;
        prof_pair(p, pc, 0, &e0, &e1);
        sk_commit none = {};
        none.first_wg = INT32_MAX;
        int e = p->L.elem == 4 ? sk_launch_attention_small(L[gi], none, (int32_t)P.work[gi].size(), st, e0, e1)
                               : sk_launch_attention(L[gi], g.v.id, (int32_t)P.work[gi].size(), st, e0, e1);
        if (e) { g_last_hip = e; return SK_E_HIP; }
        p->stats.launches++;
        wgs += (int32_t)P.work[gi].size();
        for (const sk_comb& c : P.comb[gi]) most[gi] = std::max(most[gi], c.n_parts);
        max_parts = std::max(max_parts, most[gi]);
    }
    for (int gi = 0; gi < n_groups && !P.fuse; ++gi) {
        if (P.comb[gi].empty()) continue;
        prof_pair(p, pc, 1, &e0, &e1);
        int e = sk_launch_combine(L[gi], (int32_t)P.comb[gi].size(), most[gi], Hkv, st, e0, e1);
        if (e) { g_last_hip = e; return SK_E_HIP; }
        p->stats.launches++;
    }
    p->stats.kv_bytes_streamed += P.kv_total * 2 * Hkv * p->d.head_dim * p->L.elem;
    p->last.workgroups = wgs; p->last.n_splits = max_parts; p->last.row_tiles = (int32_t)P.n_tiles;
    p->last.kernel_variant = groups[0].v.id;
    p->last.fused_merge = P.fuse ? 1 : 0;
    for (int gi = n_groups - 1; gi >= 0; --gi) if (!groups[gi].tiles.empty()) p->last.kernel_variant = groups[gi].v.id;
    return SK_OK;
}

}  // namespace

extern "C" {

size_t sk_pool_kv_bytes(const sk_pool_desc* desc)
{
    Layout L;
    if (!desc || !derive_layout(*desc, L)) return 0;
    return L.kv_bytes;
}

size_t sk_pool_workspace_bytes(const sk_pool_desc* desc)
{
    Layout L;
    if (!desc || !derive_layout(*desc, L)) return 0;
    return L.ws_bytes;
}

int sk_pool_create(const sk_pool_desc* desc, sk_pool** out)
{
    if (out) *out = nullptr;
    if (!desc || !out) return SK_E_INVAL;
    if (desc->dtype != SK_F32 && desc->dtype != SK_BF16) return SK_E_DTYPE;
    Layout L;
    if (!derive_layout(*desc, L)) return SK_E_SHAPE;
    const bool meta_only = (desc->flags & SK_POOL_METADATA_ONLY) != 0;
    if (!meta_only) {
        if (!desc->kv_mem || !desc->workspace) return SK_E_INVAL;
        if ((reinterpret_cast<uintptr_t>(desc->kv_mem) & 255) || (reinterpret_cast<uintptr_t>(desc->workspace) & 255)) return SK_E_INVAL;
        if (desc->kv_bytes < L.kv_bytes || desc->workspace_bytes < L.ws_bytes) return SK_E_WORKSPACE;
    }
    sk_pool* p = new (std::nothrow) sk_pool();
    if (!p) return SK_E_NOMEM;
    p->d = *desc;
    p->L = L;
    p->device = !meta_only;
    for (int64_t i = 0; i < desc->n_blocks; ++i) p->free_blocks.push_back((int32_t)i);
    p->refcnt.assign((size_t)desc->n_blocks, 0);
    p->sessions.resize(desc->max_sessions);
    for (int32_t i = desc->max_sessions - 1; i >= 0; --i) p->free_ids.push_back(i);
    const float scale = desc->softmax_scale != 0.f ? desc->softmax_scale : 1.0f / std::sqrt((float)desc->head_dim);
    sk_geom& g = p->geom;
    memset(&g, 0, sizeof g);
    g.kv = (const unsigned char*)desc->kv_mem;
    g.eph = meta_only ? nullptr : (const unsigned char*)desc->workspace + L.off_eph;
    g.tables = meta_only ? nullptr : (const int32_t*)((const unsigned char*)desc->workspace + L.off_tables);
    g.eph_ident = meta_only ? nullptr : (const int32_t*)((const unsigned char*)desc->workspace + L.off_ident);
    g.blk_stride = L.blk_stride; g.eph_blk_stride = L.eph_blk_stride;
    g.head_stride = L.head_stride; g.v_off = (int32_t)L.v_off;
    g.eph_head_stride = L.eph_head_stride; g.eph_v_off = (int32_t)L.eph_v_off;
    g.B = desc->block_tokens; g.log2B = ilog2_exact(desc->block_tokens);
    g.Hq = desc->n_q_heads; g.Hkv = desc->n_kv_heads; g.G = L.G; g.log2G = ilog2_exact(L.G);
    g.d = desc->head_dim; g.elem = L.elem;
    g.g_magic = (65536u + (uint32_t)L.G - 1u) / (uint32_t)L.G;
    g.scale_log2e = scale * 1.4426950408889634f;
    if (const char* t = getenv("SK_TARGET_WGS")) { int x = atoi(t); if (x > 0) { p->target_wgs = x; p->target_wgs_set = true; } }
    auto env_on = [](const char* name) { const char* x = getenv(name); return x && x[0] == '1'; };
    p->force_simple = env_on("SK_FORCE_SIMPLE");
    p->no_256 = env_on("SK_NO_256");
    p->no_small = env_on("SK_NO_SMALL");
    if (const char* t = getenv("SK_SMALL_DISTRUST")) p->distrust = atoi(t) & 3;
    p->no_pack = env_on("SK_NO_PACK");
    p->no_interleave = env_on("SK_NO_INTERLEAVE");
    p->no_stream_loads = env_on("SK_NO_STREAM_LOADS");
    p->fuse = env_on("SK_FUSE");
    p->p128 = !env_on("SK_NO_P128");
    if (const char* t = getenv("SK_P128_MIN_TOKENS")) { long long x = atoll(t); if (x >= 0) p->p128_min_tokens = x; }
    if (const char* t = getenv("SK_STREAM_MIN_TOKENS")) { long long x = atoll(t); if (x >= 0) p->stream_min_tokens = x; }
    p->fuse_list = env_on("SK_FUSE_LIST");
    p->merge_fences = env_on("SK_MERGE_FENCES");
    if (const char* t = getenv("SK_WAIT_POLLS")) { int x = atoi(t); if (x >= 0) p->wait_polls = x; }
    if (!meta_only) {
        int dev = 0, cus = 0;
        if (hipGetDevice(&dev) == hipSuccess && hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess && cus > 0)
            p->n_cus = cus;
        // Kernels read lists in it (scatter_launch) that replace those an earlier kernel read in the same place: mapped, and coherent
        // by name, as the default leaves that to HIP_HOST_COHERENT.
        hipError_t e = hipHostMalloc((void**)&p->ring, p->L.meta_bytes * kRingSlots, hipHostMallocMapped | hipHostMallocCoherent);
        if (e != hipSuccess) { g_last_hip = (int)e; delete p; return SK_E_HIP; }
        for (int i = 0; i < kRingSlots; ++i) {
            e = hipEventCreateWithFlags(&p->ring_ev[i], hipEventDisableTiming);
            if (e != hipSuccess) { g_last_hip = (int)e; sk_pool_destroy(p); return SK_E_HIP; }
        }
        // identity table over the staging blocks (one synchronous copy at creation)
        std::vector<int32_t> ident((size_t)L.eph_blocks);
        for (size_t i = 0; i < ident.size(); ++i) ident[i] = (int32_t)i;
        e = hipMemcpy((unsigned char*)desc->workspace + L.off_ident, ident.data(), ident.size() * 4, hipMemcpyHostToDevice);
        if (e != hipSuccess) { g_last_hip = (int)e; sk_pool_destroy(p); return SK_E_HIP; }
        // the merge counters start at zero; every launch leaves them at zero
        e = hipMemset((unsigned char*)desc->workspace + L.off_sync, 0, size_t(L.sync_units) * 8);
        if (e == hipSuccess) e = hipDeviceSynchronize();
        if (e != hipSuccess) { g_last_hip = (int)e; sk_pool_destroy(p); return SK_E_HIP; }
    }
    *out = p;
    return SK_OK;
}

int sk_pool_destroy(sk_pool* p)
{
    if (!p) return SK_E_INVAL;
    if (p->device) {
        for (int i = 0; i < kRingSlots; ++i)
            if (p->ring_ev[i]) (void)hipEventDestroy(p->ring_ev[i]);
        for (sk_pool::ProfRec& r : p->prof) { (void)hipEventDestroy(r.start); (void)hipEventDestroy(r.stop); }
        if (p->ring) (void)hipHostFree(p->ring);
    }
    delete p;
    return SK_OK;
}

int sk_pool_blocks_free(const sk_pool* p, int64_t* out)
{
    if (!p || !out) return SK_E_INVAL;
    *out = (int64_t)p->free_blocks.size();
    return SK_OK;
}

int sk_pool_set_alloc_order(sk_pool* p, const int32_t* perm, int64_t n)
{
    if (!p || !perm || n != p->d.n_blocks) return SK_E_INVAL;
    if (p->blocks_in_use != 0) return SK_E_INVAL;
    std::vector<char> seen((size_t)n, 0);
    for (int64_t i = 0; i < n; ++i) {
        if (perm[i] < 0 || perm[i] >= n || seen[perm[i]]) return SK_E_INVAL;
        seen[perm[i]] = 1;
    }
    p->free_blocks.assign(perm, perm + n);
    return SK_OK;
}

int sk_session_create(sk_pool* p, int32_t* out_id)
{
    if (!p || !out_id) return SK_E_INVAL;
    if (p->free_ids.empty()) return SK_E_NOMEM;
    int32_t id = p->free_ids.back();
    p->free_ids.pop_back();
    Session& s = p->sessions[id];
    s.live = true; s.len = 0; s.frozen = 0; s.win = 0; s.blocks.clear(); s.may_share = false;
    *out_id = id;
    return SK_OK;
}

int sk_session_destroy(sk_pool* p, int32_t id)
{
    Session* s = get_session(p, id);
    if (!s) return p ? SK_E_BADSESSION : SK_E_INVAL;
    for (int32_t b : s->blocks) release_block(p, b);
    s->blocks.clear(); s->len = 0; s->frozen = 0; s->win = 0; s->live = false;
    p->free_ids.push_back(id);
    return SK_OK;
}

int sk_session_length(const sk_pool* p, int32_t id, int64_t* out)
{
    const Session* s = get_session(p, id);
    if (!p || !out) return SK_E_INVAL;
    if (!s) return SK_E_BADSESSION;
    *out = s->retained();
    return SK_OK;
}

int sk_session_block_table(const sk_pool* p, int32_t id, const int32_t** table, int64_t* n_blocks)
{
    const Session* s = get_session(p, id);
    if (!p || !table || !n_blocks) return SK_E_INVAL;
    if (!s) return SK_E_BADSESSION;
    *table = s->blocks.data();
    *n_blocks = (int64_t)s->blocks.size();
    return SK_OK;
}

int sk_session_append(sk_pool* p, int32_t id, const void* q, const void* k, const void* v, int32_t L,
                      void* out, int out_dtype, float* lse, void* hip_stream)
{
    if (!p) return SK_E_INVAL;
    Session* s = get_session(p, id);
    if (!s) return SK_E_BADSESSION;
    if (L < 0) return SK_E_INVAL;
    if (L == 0) return SK_OK;
    if (L > p->L.max_batch_tokens) return SK_E_WORKSPACE;
    if (p->device) {
        if (!k || !v || (!q) != (!out)) return SK_E_INVAL;
        if (!aligned16(q) || !aligned16(k) || !aligned16(v) || !aligned16(out) || !aligned16(lse)) return SK_E_INVAL;
        if (q) { int rc = check_out_dtype(p, out_dtype); if (rc) return rc; }
    }
    if (s->len + L > p->L.max_session_tokens) return SK_E_NOMEM;
    const int64_t need = blocks_needed(p, s->len, L);
    if (need + (tail_shared(p, s) ? 1 : 0) > (int64_t)p->free_blocks.size()) return SK_E_NOMEM;
    // everything else that can refuse the call, before it changes anything: the decomposition of the
    // attention, and the ring slot of a scatter list too long for the kernel arguments
    hipStream_t st = (hipStream_t)hip_stream;
    const int64_t n = s->len;
    const bool attend = p->device ? q != nullptr : true;
    RegPlan plan;
    if (attend) {
        Variant v;
        const bool small = (pick_variant(p, L, v, false, n) && v.id == SK_KV_SMALL) || p->L.elem == 4;      // attends to the chunk where it lies
        int rc = plan_regular(p, id, L, (int32_t)n, small ? n : n + L, small ? L : 0, 0, s->frozen, s->win, 0, plan);
        if (rc) return rc;
    }
    const bool in_place = attend && plan.L.own_mode != SK_OWN_NONE;
    const bool one_launch = in_place && scatter_groups(n, L) <= SK_COMMIT_ITEMS;      // the attention launch commits too
    ScatterSlot ss;
    { int rc = scatter_reserve(p, scatter_groups(n, L), ss); if (rc) return rc; }
    if (in_place && p->device && results_over_own(p, L, k, v, out, out_dtype, lse)) { int rc = copy_own(p, L, &k, &v, st); if (rc) return rc; }
    // from here on only a failing HIP call can stop the call; what it changed is taken back
    Undo u;
    int64_t first_new = 0;
    { int rc = grow_session(p, s, L, u, &first_new, st); if (rc) return rc; }
    std::vector<sk_scatter> items;
    build_scatter(p, s, id, n, 0, L, first_new, false, 0, items);
    int rc;
    if (in_place) { plan.own_k = k; plan.own_v = v; }
    if (one_launch) {
        plan.commit_items = (int32_t)items.size();
        memcpy(plan.commit.item, items.data(), items.size() * sizeof(sk_scatter));
        rc = inject(p, SK_SITE_SCATTER) ? SK_E_HIP : SK_OK;
    } else rc = scatter_launch(p, ss, items, k, v, st);
    if (rc) { rollback(p, u, false); return rc; }
    if (attend) {
        rc = launch_regular(p, plan, q, out, out_dtype, lse, st);
        if (rc) { rollback(p, u, !one_launch || plan.enqueued); return rc; }
    }
    p->stats.tokens_appended += L;
    return SK_OK;
}

int sk_session_query(sk_pool* p, int32_t id, const void* q, const void* k, const void* v, int32_t nq,
                     void* out, int out_dtype, float* lse, int32_t n_splits, void* hip_stream)
{
    if (!p) return SK_E_INVAL;
    Session* s = get_session(p, id);
    if (!s) return SK_E_BADSESSION;
    if (nq < 0 || n_splits < 0) return SK_E_INVAL;
    if (nq == 0) return SK_OK;
    if (!p->device) return SK_E_NODEVICE;
    if (!q || !out || (!k) != (!v)) return SK_E_INVAL;
    if (!aligned16(q) || !aligned16(k) || !aligned16(v) || !aligned16(out) || !aligned16(lse)) return SK_E_INVAL;
    int rc = check_out_dtype(p, out_dtype);
    if (rc) return rc;
    if (nq > p->L.max_batch_tokens) return SK_E_WORKSPACE;
    if (!k && s->retained() == 0) return SK_E_EMPTY;
    Variant vv;
    if (!pick_variant(p, nq, vv)) return SK_E_SHAPE;
    hipStream_t st = (hipStream_t)hip_stream;
    RegPlan plan;
    if (k) rc = plan_regular(p, id, nq, (int32_t)s->len, s->len, nq, (int32_t)s->len, s->frozen, s->win, n_splits, plan);
    else rc = plan_regular(p, id, nq, SK_NO_CAUSAL, s->len, 0, 0, s->frozen, s->win, n_splits, plan);
    if (rc) return rc;
    // Own K/V are read where they lie, or staged by the attention kernel: with one row tile per KV head one workgroup of
    // each head attends to them, and up to 64 tokens take it less time than the others their keys.
    const bool in_place = plan.L.own_mode != SK_OWN_NONE;
    const bool over = k && results_over_own(p, nq, k, v, out, out_dtype, lse);
    const bool stages = !in_place && !over && plan.L.n_tiles == 1 && plan.v.id != SK_KV_SIMPLE && nq <= SK_STAGE_TOKENS;
    if (k && stages && inject(p, SK_SITE_SCATTER)) return SK_E_HIP;
    if (in_place && over) { rc = copy_own(p, nq, &k, &v, st); if (rc) return rc; }
    if (k && (in_place || stages)) { plan.own_k = k; plan.own_v = v; }
    else if (k) {
        ScatterSlot ss;
        rc = scatter_reserve(p, scatter_groups(0, nq), ss);
        if (rc) return rc;
        std::vector<sk_scatter> items;
        build_scatter(p, nullptr, id, 0, 0, nq, 0, true, 0, items);
        rc = scatter_launch(p, ss, items, k, v, st);
        if (rc) return rc;
    }
    rc = launch_regular(p, plan, q, out, out_dtype, lse, st);
    if (rc) return rc;
    p->stats.tokens_queried += nq;
    return SK_OK;
}

int sk_batch_step(sk_pool* p, int32_t n_items, const int32_t* session_id, const int32_t* op, const int32_t* cu_tokens,
                  const void* q, const void* k, const void* v, void* out, int out_dtype, float* lse, void* hip_stream)
{
    if (!p || n_items < 0) return SK_E_INVAL;
    if (n_items == 0) return SK_OK;
    if (!session_id || !op || !cu_tokens) return SK_E_INVAL;
    if (n_items > p->d.max_sessions) return SK_E_INVAL;        // sessions are distinct
    if (cu_tokens[0] != 0) return SK_E_INVAL;
    std::vector<char> seen((size_t)p->d.max_sessions, 0);
    int64_t need_blocks = 0;
    bool any_kv = false;
    std::vector<char> shared((size_t)n_items, 0);               // as it is before an append takes its own copy of a shared tail
    for (int i = 0; i < n_items; ++i) {
        const Session* s = get_session(p, session_id[i]);
        if (!s) return SK_E_BADSESSION;
        if (seen[session_id[i]]) return SK_E_INVAL;
        seen[session_id[i]] = 1;
        const int64_t T = int64_t(cu_tokens[i + 1]) - cu_tokens[i];
        if (T < 0) return SK_E_INVAL;
        if (op[i] != SK_OP_APPEND && op[i] != SK_OP_QUERY_A && op[i] != SK_OP_QUERY_B) return SK_E_INVAL;
        if (T == 0) continue;
        shared[(size_t)i] = holds_shared(p, *s);
        if (op[i] == SK_OP_APPEND) {
            if (s->len + T > p->L.max_session_tokens) return SK_E_NOMEM;
            need_blocks += blocks_needed(p, s->len, T) + (tail_shared(p, s) ? 1 : 0);
        }
        if (op[i] == SK_OP_QUERY_A && s->retained() == 0) return SK_E_EMPTY;
        if (op[i] != SK_OP_QUERY_A) any_kv = true;
    }
    const int64_t total = cu_tokens[n_items];
    if (total > p->L.max_batch_tokens) return SK_E_WORKSPACE;
    if (need_blocks > (int64_t)p->free_blocks.size()) return SK_E_NOMEM;
    {   // staging blocks of the queries that bring their own K/V
        int64_t eph_need = 0;
        for (int i = 0; i < n_items; ++i)
            if (op[i] == SK_OP_QUERY_B) eph_need += (int64_t(cu_tokens[i + 1]) - cu_tokens[i] + 15) / 16;
        if (eph_need > p->L.eph_blocks) return SK_E_WORKSPACE;
    }
    if (p->device) {
        if (!q || !out || (any_kv && (!k || !v))) return SK_E_INVAL;
        if (!aligned16(q) || !aligned16(k) || !aligned16(v) || !aligned16(out) || !aligned16(lse)) return SK_E_INVAL;
        int rc = check_out_dtype(p, out_dtype);
        if (rc) return rc;
        Variant vv;
        if (!pick_variant(p, 1, vv)) return SK_E_SHAPE;
    }
    // From here on the sessions change; whatever stops the call afterwards (the lists do not fit the
    // workspace, a HIP call fails) takes every change back, in reverse order.
    ScatterBatch sb;
    sb.k = k; sb.v = v;
    ListGroup groups[3];
    const bool allow_256 = !p->no_256;
    struct Item { TileReq base; int32_t row0, tokens; };
    std::vector<Item> tall;                 // head_dim 64: the items in 256-row tiles
    int64_t eph_cursor = 0;
    std::vector<Undo> undo;
    int64_t appended = 0, queried = 0;
    auto take_back = [&](bool keep_copies) {
        for (size_t i = undo.size(); i-- > 0;) rollback(p, undo[i], keep_copies);
    };
    hipStream_t st = (hipStream_t)hip_stream;
    for (int i = 0; i < n_items; ++i) {
        Session* s = get_session(p, session_id[i]);
        const int32_t T = cu_tokens[i + 1] - cu_tokens[i];
        if (T == 0) continue;
        const int32_t id = session_id[i];
        const int64_t n = s->len;
        const int32_t tbl_off = int32_t(int64_t(id) * p->L.max_blocks_per_session);
        TileReq base = {};
        base.tbl_off = tbl_off;
        base.hole_lo = (int32_t)s->frozen; base.hole_hi = (int32_t)s->win;
        base.alone = 1; base.shared = shared[(size_t)i];        // (sessions are distinct, but forks share the blocks of a prefix)
        if (op[i] == SK_OP_APPEND) {
            Undo u;
            int64_t first_new = 0;
            int rc = grow_session(p, s, T, u, &first_new, st);
            if (rc) { take_back(false); return rc; }
            undo.push_back(u);
            appended += T;
            build_scatter(p, s, id, n, cu_tokens[i], T, first_new, false, 0, sb.items);
            base.pos0 = (int32_t)n; base.kv_vis = int32_t(n + T);
        } else {
            queried += T;
            if (op[i] == SK_OP_QUERY_B) {
                build_scatter(p, nullptr, id, 0, cu_tokens[i], T, 0, true, eph_cursor, sb.items);
                base.pos0 = (int32_t)n; base.kv_vis = (int32_t)n;
                base.eph_blk[0] = (int32_t)eph_cursor; base.eph_cnt[0] = T; base.eph_pos0[0] = (int32_t)n;
                eph_cursor += (T + 15) / 16;
            } else {
                base.pos0 = SK_NO_CAUSAL; base.kv_vis = (int32_t)n;
            }
        }
        // items of more than 128 rows per KV head (the appends) go to the 256-row kernel, which is
        // launched first; then the 128-row items, then the small ones
        Variant vv;
        if (!pick_variant(p, T, vv, allow_256)) { take_back(false); return SK_E_SHAPE; }
        ListGroup& g = groups[vv.id == SK_KV_MFMA64 ? 2 : vv.id == SK_KV_MFMA128 ? 1 : 0];
        g.v = vv; g.q = q; g.out = out; g.lse = lse;
        add_tiles(g, base, cu_tokens[i], T);
        if (vv.id == SK_KV_MFMA256 && list_narrow(p, vv)) tall.push_back({base, cu_tokens[i], T});
    }
    if (list_narrow(p, groups[0].v) && !groups[0].tiles.empty()) {
        // head_dim 64: the items above 128 rows in tiles of 128, together with those of 65 to 128, where that is expected to end
        // earlier.  us per step in 256-row tiles and in 128: 12 sessions of 32/8 heads, 137 tokens at 888 cached each, 68 and 55; 48 of
        // 14/2, 84 at 10,615, 307 and 256; 4 of 12/4, 292 at
        // 15,626, 112 and 166.  348 random steps against 128-row tiles always: with 256-row ones always 0.90 of the time in the
        // geometric mean, 48 more than 3 % slower and up to 33; by expected end 0.81, the slowest 2 %.  Lists beyond 16 KiB count the
        // 2 us that they take longer: 400 of the steps in list_chunk's comment then take 0.887 of their former time, with 14 here 0.902, with
        // nothing 0.874 and one of them 1.4 times as long.
        constexpr double kCarriedUs = 2.0;
        ListGroup low = groups[1];
        low.v = Variant{SK_KV_MFMA128, 128, 128 / p->L.G};
        low.q = q; low.out = out; low.lse = lse;
        for (const Item& it : tall) add_tiles(low, it.base, it.row0, it.tokens);
        const size_t scatter = sb.items.size() * sizeof(sk_scatter);
        const ListGroup* const as_low[2] = {&low, &groups[2]};
        const ListGroup* const as_tall[3] = {&groups[0], &groups[1], &groups[2]};
        const double tall_us = list_cost(p, as_tall, 3, scatter, kCarriedUs);
        if (list_cost(p, as_low, 2, scatter, kCarriedUs, tall_us) < tall_us) {
            groups[0].tiles.clear();
            groups[1] = std::move(low);
        }
    }
    ListPlan plan;
    int rc = plan_list(p, &sb, 1, groups, 3, plan);
    if (rc) { take_back(false); return rc; }
    rc = launch_list(p, plan, &sb, 1, groups, 3, out_dtype, st);
    if (rc) { take_back(plan.scatter_enqueued); return rc; }
    p->stats.tokens_appended += appended;
    p->stats.tokens_queried += queried;
    return SK_OK;
}

int sk_session_query_shared_prefix(sk_pool* p, int32_t id, const void* qp, const void* kp, const void* vp, int32_t P,
                                   const void* qs, const void* ks, const void* vs, int32_t NQ, int32_t Sfx,
                                   void* out_prefix, void* out_suffix, int out_dtype,
                                   float* lse_prefix, float* lse_suffix, void* hip_stream)
{
    if (!p) return SK_E_INVAL;
    Session* s = get_session(p, id);
    if (!s) return SK_E_BADSESSION;
    if (P < 0 || NQ < 0 || Sfx < 0) return SK_E_INVAL;
    if (P == 0 && (NQ == 0 || Sfx == 0)) return SK_OK;
    if (!p->device) return SK_E_NODEVICE;
    if (P > 0 && (!qp || !kp || !vp || !out_prefix)) return SK_E_INVAL;
    const bool has_sfx = NQ > 0 && Sfx > 0;
    if (has_sfx && (!qs || !ks || !vs || !out_suffix)) return SK_E_INVAL;
    if (!aligned16(qp) || !aligned16(kp) || !aligned16(vp) || !aligned16(qs) || !aligned16(ks) || !aligned16(vs) ||
        !aligned16(out_prefix) || !aligned16(out_suffix) || !aligned16(lse_prefix) || !aligned16(lse_suffix)) return SK_E_INVAL;
    int rc = check_out_dtype(p, out_dtype);
    if (rc) return rc;
    const int64_t total = int64_t(P) + (has_sfx ? int64_t(NQ) * Sfx : 0);
    const int64_t sfx_blocks = (Sfx + 15) / 16, pre_blocks = (P + 15) / 16;
    if (total > p->L.max_batch_tokens || pre_blocks + (has_sfx ? NQ * sfx_blocks : 0) > p->L.eph_blocks) return SK_E_WORKSPACE;
    Variant vtest;
    if (!pick_variant(p, 1, vtest)) return SK_E_SHAPE;
    const int64_t n = s->len;
    const int32_t tbl_off = int32_t(int64_t(id) * p->L.max_blocks_per_session);
    ScatterBatch sb[2];
    ListGroup groups[2];
    if (P > 0) {
        sb[0].k = kp; sb[0].v = vp;
        build_scatter(p, nullptr, id, 0, 0, P, 0, true, 0, sb[0].items);
        TileReq base = {};
        base.tbl_off = tbl_off; base.pos0 = (int32_t)n; base.kv_vis = (int32_t)n;
        base.hole_lo = (int32_t)s->frozen; base.hole_hi = (int32_t)s->win;
        base.eph_blk[0] = 0; base.eph_cnt[0] = P; base.eph_pos0[0] = (int32_t)n;
        pick_variant(p, P, groups[0].v);
        groups[0].q = qp; groups[0].out = out_prefix; groups[0].lse = lse_prefix;
        add_tiles(groups[0], base, 0, P);
    }
    if (has_sfx) {
        sb[1].k = ks; sb[1].v = vs;
        pick_variant(p, Sfx, groups[1].v);
        groups[1].q = qs; groups[1].out = out_suffix; groups[1].lse = lse_suffix;
        // Short suffixes are packed: several questions share one 256-row tile of the eight-wave
        // kernel (their rows see the same cache and prefix; each sees its own suffix), when a
        // question's rows are a multiple of a wave's 32 and divide 256.
        const int64_t rows_q = int64_t(Sfx) * p->L.G;
        const bool can_pack = groups[1].v.id != SK_KV_SIMPLE && rows_q < 256 && rows_q % 32 == 0 &&
                              256 % rows_q == 0 && NQ > 1 && !p->no_pack;
        for (int32_t j = 0; j < NQ; ++j)
            build_scatter(p, nullptr, id, 0, j * Sfx, Sfx, 0, true, pre_blocks + j * sfx_blocks, sb[1].items);
        auto cut = [&](ListGroup& g, bool pack) {
            const int32_t per_tile = pack ? int32_t(256 / rows_q) : 1;
            if (pack) g.v = Variant{SK_KV_MFMA256, 256, 256 / p->L.G};
            for (int32_t j = 0; j < NQ; j += per_tile) {
                const int32_t nq_tile = std::min(per_tile, NQ - j);
                TileReq base = {};
                base.tbl_off = tbl_off; base.pos0 = int32_t(n + P); base.kv_vis = (int32_t)n;
                base.hole_lo = (int32_t)s->frozen; base.hole_hi = (int32_t)s->win;
                base.eph_blk[0] = 0; base.eph_cnt[0] = P; base.eph_pos0[0] = (int32_t)n;
                base.eph_blk[1] = int32_t(pre_blocks + j * sfx_blocks); base.eph_cnt[1] = Sfx; base.eph_pos0[1] = int32_t(n + P);
                if (pack) {
                    base.tok_period = Sfx; base.sub_blocks = (int32_t)sfx_blocks;
                    base.q_tok0 = j * Sfx; base.n_tok = nq_tile * Sfx;
                    g.tiles.push_back(base);
                } else add_tiles(g, base, j * Sfx, Sfx);
            }
        };
        // head_dim 64 packs where that is expected to end earlier: a tile walks the suffixes of all its questions, one after the
        // other.  us per batch, one question a tile and packed: 8 questions of 32 tokens at 162 cached (8/8 heads) 31 and 48, 43 of 8 at
        // 957 (32/8) 58 and 75; 5 of 8 behind a prefix of 16 at 1,550 51 and 47.  200 random batches against no packing: packed always
        // 0.91 of the time, 50 more than 3 % slower and up to 56; by expected end 0.82, 4 more than 3 % slower, up to 14.  That was with
        // 14 us for lists beyond 16 KiB, and is kept for this choice: it leaves to the packed tiles what they save in lists and launches
        // (300 random batches without it: 1.2 % less time in the geometric mean, two more than 3 % slower).
        constexpr double kListsUs = 14.0;
        if (can_pack && list_narrow(p, groups[1].v)) {
            ListGroup apart = groups[1];
            cut(apart, false);
            cut(groups[1], true);
            const size_t scatter = (sb[0].items.size() + sb[1].items.size()) * sizeof(sk_scatter);
            const ListGroup* const as_apart[2] = {&groups[0], &apart};
            const ListGroup* const as_packed[2] = {&groups[0], &groups[1]};
            const double packed_us = list_cost(p, as_packed, 2, scatter, kListsUs);
            if (list_cost(p, as_apart, 2, scatter, kListsUs, packed_us) < packed_us) groups[1] = std::move(apart);
        } else cut(groups[1], can_pack);
    }
    ListPlan plan;
    rc = plan_list(p, sb, 2, groups, 2, plan);
    if (rc) return rc;
    rc = launch_list(p, plan, sb, 2, groups, 2, out_dtype, (hipStream_t)hip_stream);
    if (rc) return rc;
    p->stats.tokens_queried += total;
    return SK_OK;
}

int sk_session_gather(const sk_pool* p, int32_t id, int64_t first, int64_t count, void* k_out, void* v_out, void* hip_stream)
{
    if (!p) return SK_E_INVAL;
    const Session* s = get_session(p, id);
    if (!s) return SK_E_BADSESSION;
    if (!p->device) return SK_E_NODEVICE;
    if (first < 0 || count < 0 || first + count > s->retained()) return SK_E_INVAL;
    if (count == 0) return SK_OK;
    if (!k_out || !v_out || !aligned16(k_out) || !aligned16(v_out)) return SK_E_INVAL;
    // retained tokens [first, first+count) = a piece of [0, frozen) followed by a piece of [win, len)
    const int32_t tbl_off = int32_t(int64_t(id) * p->L.max_blocks_per_session);
    const int64_t row_bytes = int64_t(p->d.n_kv_heads) * p->d.head_dim * p->L.elem;
    const int64_t n_a = std::max<int64_t>(0, std::min(first + count, s->frozen) - first);
    if (n_a > 0) {
        int e = sk_launch_gather(p->geom, tbl_off, first, n_a, k_out, v_out, hip_stream);
        if (e) { g_last_hip = e; return SK_E_HIP; }
    }
    if (count > n_a) {
        const int64_t first_b = std::max(first, s->frozen) - s->frozen + s->win;
        int e = sk_launch_gather(p->geom, tbl_off, first_b, count - n_a, (unsigned char*)k_out + n_a * row_bytes,
                                 (unsigned char*)v_out + n_a * row_bytes, hip_stream);
        if (e) { g_last_hip = e; return SK_E_HIP; }
    }
    return SK_OK;
}

int sk_session_truncate(sk_pool* p, int32_t id, int64_t new_length)
{
    if (!p) return SK_E_INVAL;
    Session* s = get_session(p, id);
    if (!s) return SK_E_BADSESSION;
    if (new_length < 0 || new_length > s->retained()) return SK_E_INVAL;
    if (new_length <= s->frozen) { s->frozen = new_length; s->win = new_length; s->len = new_length; }
    else s->len = s->win + (new_length - s->frozen);
    const int64_t B = p->d.block_tokens;
    const size_t keep = size_t((s->len + B - 1) / B);
    while (s->blocks.size() > keep) {
        release_block(p, s->blocks.back());
        s->blocks.pop_back();
    }
    return SK_OK;
}

int sk_session_freeze(sk_pool* p, int32_t id, int64_t n_frozen)
{
    if (!p) return SK_E_INVAL;
    Session* s = get_session(p, id);
    if (!s) return SK_E_BADSESSION;
    if (s->win != s->frozen) return SK_E_INVAL;           // tokens behind the frozen region were already evicted
    if (n_frozen < s->frozen || n_frozen > s->len) return SK_E_INVAL;
    s->frozen = n_frozen; s->win = n_frozen;
    return SK_OK;
}

int sk_session_evict_oldest(sk_pool* p, int32_t id, int64_t n_tokens, void* hip_stream)
{
    if (!p) return SK_E_INVAL;
    Session* s = get_session(p, id);
    if (!s) return SK_E_BADSESSION;
    if (n_tokens < 0 || n_tokens > s->len - s->win) return SK_E_INVAL;
    if (n_tokens == 0) return SK_OK;
    // blocks that lie entirely inside the hole go back to the pool; storage indices behind them move down
    const int64_t B = p->d.block_tokens;
    const int64_t win = s->win + n_tokens;
    const int64_t b0 = (s->frozen + B - 1) / B, b1 = win / B;
    if (b1 <= b0) {                  // no whole block is freed: the window start moves, nothing else
        s->win = win;
        p->stats.tokens_evicted += n_tokens;
        return SK_OK;
    }
    // The moved tail of the session's device block table is rewritten (ordered on the caller's
    // stream); the host side changes only once that copy is enqueued, so a failure leaves the
    // session as it was.
    const size_t n_moved = s->blocks.size() - (size_t)b1;
    if (n_moved > 0) {
        int slot; unsigned char* host;
        int rc = ring_acquire(p, &slot, &host);
        if (rc) return rc;
        const size_t bytes = n_moved * sizeof(int32_t);
        if (host) memcpy(host, s->blocks.data() + b1, bytes);
        int32_t* dev_tbl = p->device ? (int32_t*)((unsigned char*)p->d.workspace + p->L.off_tables) + int64_t(id) * p->L.max_blocks_per_session + b0
                                     : nullptr;
        rc = ring_copy(p, slot, dev_tbl, bytes, (hipStream_t)hip_stream);
        if (rc) return rc;
    }
    const int64_t k = b1 - b0;
    for (int64_t b = b0; b < b1; ++b) release_block(p, s->blocks[(size_t)b]);
    s->blocks.erase(s->blocks.begin() + b0, s->blocks.begin() + b1);
    s->win = win - k * B; s->len -= k * B;
    p->stats.tokens_evicted += n_tokens;
    return SK_OK;
}

int sk_session_fork(sk_pool* p, int32_t src_id, int64_t n_prefix, int32_t* out_id, void* hip_stream)
{
    if (!p || !out_id) return SK_E_INVAL;
    Session* src = get_session(p, src_id);
    if (!src) return SK_E_BADSESSION;
    if (n_prefix < 0 || n_prefix > src->retained()) return SK_E_INVAL;
    if (p->free_ids.empty()) return SK_E_NOMEM;
    // storage layout of the new session: the same hole as the source if the prefix reaches behind it
    const int64_t B = p->d.block_tokens;
    int64_t frozen, win, len;
    if (n_prefix <= src->frozen) frozen = win = len = n_prefix;
    else { frozen = src->frozen; win = src->win; len = src->win + (n_prefix - src->frozen); }
    const int64_t n_blk = (len + B - 1) / B;
    const bool tail_partial = len % B != 0;      // the new session will write into its last block: it gets a copy
    if (tail_partial && p->free_blocks.empty()) return SK_E_NOMEM;
    const int32_t id = p->free_ids.back();
    std::vector<int32_t> blocks(src->blocks.begin(), src->blocks.begin() + n_blk);
    int32_t tail_src = -1;
    if (tail_partial) { tail_src = blocks.back(); blocks.back() = p->free_blocks.front(); }
    // Device work first (the new session's block table, then the copy of the partly filled last block,
    // all KV heads), into places no live session reads; the host side changes only when both are
    // enqueued, so a failure leaves the pool as it was.
    hipStream_t st = (hipStream_t)hip_stream;
    if (n_blk > 0) {
        int slot; unsigned char* host;
        int rc = ring_acquire(p, &slot, &host);
        if (rc) return rc;
        const size_t bytes = (size_t)n_blk * sizeof(int32_t);
        if (host) memcpy(host, blocks.data(), bytes);
        int32_t* dev_tbl = p->device ? (int32_t*)((unsigned char*)p->d.workspace + p->L.off_tables) + int64_t(id) * p->L.max_blocks_per_session
                                     : nullptr;
        rc = ring_copy(p, slot, dev_tbl, bytes, st);
        if (rc) return rc;
        if (tail_partial) {
            if (inject(p, SK_SITE_BLOCK_COPY)) return SK_E_HIP;
            if (p->device) {
                int e = sk_launch_copy_block(p->geom, (unsigned char*)p->d.kv_mem, tail_src, blocks.back(), st);
                if (e) { g_last_hip = e; return SK_E_HIP; }
            }
        }
    }
    p->free_ids.pop_back();
    Session& d = p->sessions[id];
    d.live = true; d.frozen = frozen; d.win = win; d.len = len;
    src->may_share = d.may_share = true;
    d.blocks.swap(blocks);
    for (int64_t i = 0; i < n_blk - (tail_partial ? 1 : 0); ++i) p->refcnt[(size_t)d.blocks[(size_t)i]]++;
    if (tail_partial) {
        p->refcnt[(size_t)d.blocks.back()] = 1;
        p->free_blocks.pop_front();
        p->blocks_in_use++;
    }
    *out_id = id;
    p->stats.forks++;
    return SK_OK;
}

int sk_pool_inject_failure(sk_pool* p, int32_t site, int32_t countdown)
{
    if (!p || site < 0 || site > SK_SITE_PLAN || countdown < 0) return SK_E_INVAL;
    p->inject_site = countdown > 0 ? site : 0;
    p->inject_countdown = countdown;
    return SK_OK;
}

int sk_pool_set_profiling(sk_pool* p, int enable)
{
    if (!p || !p->device) return p ? SK_E_NODEVICE : SK_E_INVAL;
    p->profiling = enable != 0;
    return SK_OK;
}

int sk_pool_read_profile(sk_pool* p, sk_profile* out, float* attn_pc, float* comb_pc, int32_t capacity)
{
    if (!p || !out) return SK_E_INVAL;
    out->calls = p->prof_calls; out->attention_ms = 0; out->combine_ms = 0;
    for (int32_t i = 0; i < p->prof_calls && i < capacity; ++i) {
        if (attn_pc) attn_pc[i] = 0.f;
        if (comb_pc) comb_pc[i] = 0.f;
    }
    int rc = SK_OK;
    for (size_t i = 0; i < p->prof_used && rc == SK_OK; ++i) {
        const sk_pool::ProfRec& r = p->prof[i];
        float ms = 0.f;
        if (hipEventSynchronize(r.stop) != hipSuccess || hipEventElapsedTime(&ms, r.start, r.stop) != hipSuccess) { rc = SK_E_HIP; break; }
        if (r.kind == 0) { out->attention_ms += ms; if (attn_pc && r.call < capacity) attn_pc[r.call] += ms; }
        else { out->combine_ms += ms; if (comb_pc && r.call < capacity) comb_pc[r.call] += ms; }
    }
    p->prof_used = 0; p->prof_calls = 0;
    return rc;
}

int64_t sk_pool_element_offset(const sk_pool* p, int64_t block, int32_t kv_head, int32_t is_v, int32_t slot, int32_t dim)
{
    if (!p || block < 0 || block >= p->d.n_blocks || kv_head < 0 || kv_head >= p->d.n_kv_heads ||
        slot < 0 || slot >= p->d.block_tokens || dim < 0 || dim >= p->d.head_dim) return -1;
    int64_t off = block * p->L.blk_stride + int64_t(kv_head) * p->L.head_stride;
    if (!is_v) return off + (int64_t(slot) * p->d.head_dim + dim) * p->L.elem;
    off += p->L.v_off;
    if (p->d.dtype == SK_BF16) return off + ((int64_t(slot >> 4) * p->d.head_dim + dim) * 16 + (slot & 15)) * p->L.elem;
    return off + (int64_t(slot) * p->d.head_dim + dim) * p->L.elem;
}

int sk_pool_get_stats(const sk_pool* p, sk_pool_stats* out)
{
    if (!p || !out) return SK_E_INVAL;
    *out = p->stats;
    return SK_OK;
}

int sk_pool_last_launch(const sk_pool* p, sk_launch_info* out)
{
    if (!p || !out) return SK_E_INVAL;
    *out = p->last;
    return SK_OK;
}

const char* sk_strerror(int status)
{
    switch (status) {
    case SK_OK: return "ok";
    case SK_E_INVAL: return "invalid argument";
    case SK_E_SHAPE: return "unsupported shape";
    case SK_E_DTYPE: return "unsupported element type";
    case SK_E_NOMEM: return "pool exhausted";
    case SK_E_BADSESSION: return "no such session";
    case SK_E_EMPTY: return "softmax over zero keys";
    case SK_E_WORKSPACE: return "buffer too small for this call";
    case SK_E_HIP: return "HIP runtime error";
    case SK_E_NODEVICE: return "metadata-only pool";
    default: return "unknown status";
    }
}

int sk_last_hip_error(void) { return g_last_hip; }
int sk_version(void) { return 2; }

}  // extern "C"
