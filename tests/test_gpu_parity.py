"""GPU parity: the HIP path (through the C ABI) against the fp64 oracle, element by element, on
the same seeded inputs.  Sizes span several key tiles, several row tiles and ragged tails."""
import numpy as np
import pytest
import torch

import paper_2605_13784_amd as sk
from workloads import synth
from gpu_common import Pair, compare, dev

pytestmark = pytest.mark.gpu


def test_cfg1_fp32_single_session_every_step():
    """Workload 1: fp32, 4/4 heads, d=64; 16 appends of 64 tokens to 1,024 cached tokens, then 4
    non-committing queries of 16 tokens (cache-only and with own K/V); parity on every step."""
    shape = synth.CFG1
    gen = synth.generator(1)
    pr = Pair(shape, block_tokens=16, n_blocks=80, kv_fill=0xFF)       # 0xFF bytes = NaN canaries
    sid = pr.create()
    for step in range(16):
        q, k, v = synth.draw_qkv(gen, 64, shape)
        pr.append(sid, q, k, v, name="cfg1 append %d" % step)
    pr.check_cache(sid)
    before = pr.pool.kv_mem.clone()
    for i in range(4):
        q, k, v = synth.draw_qkv(gen, 16, shape)
        pr.query(sid, q, name="cfg1 query A %d" % i)
        pr.query(sid, q, k, v, name="cfg1 query B %d" % i)
        pr.query(sid, q, n_splits=3, name="cfg1 query A splits=3 %d" % i)
    torch.cuda.synchronize()
    assert torch.equal(before, pr.pool.kv_mem)
    assert pr.pool.sk_session_length(sid) == 1024


# the instances and the cache policy that the library keeps for long caches, taken at any length
LONG_CACHE_PATHS = {"SK_P128_MIN_TOKENS": "0", "SK_STREAM_MIN_TOKENS": "0"}


@pytest.mark.parametrize("block_tokens,env", [(16, None), (64, None), (16, LONG_CACHE_PATHS)])
def test_bf16_gqa_ragged_appends_and_queries(block_tokens, env):
    """Llama-3-8B-shaped layer (32/8 heads, d=128, bf16) at a size the oracle finishes in seconds:
    appends of ragged lengths (several row tiles, partial tiles, single tokens, block-straddling),
    then queries of several lengths in both modes with several split counts; once more with the
    eight-wave 128-row instance and the non-temporal loads that single-session calls of 65-128 rows
    otherwise only take from 512 keys a workgroup / 65,536 cached tokens on."""
    shape = synth.CFG2
    gen = synth.generator(2, stream=1)
    pr = Pair(shape, block_tokens=block_tokens, n_blocks=4096 // block_tokens + 8, kv_fill=0xFF, max_batch_tokens=1024, env=env)
    sid = pr.create()
    for i, L in enumerate([256, 100, 7, 1, 333, 64, 15, 1000]):
        q, k, v = synth.draw_qkv(gen, L, shape)
        pr.append(sid, q, k, v, name="append %d (L=%d)" % (i, L))
    pr.check_cache(sid)
    n = pr.pool.sk_session_length(sid)
    assert n == 1776
    before = pr.pool.kv_mem.clone()
    for nq in [32, 16, 1, 5, 64, 100]:
        q, k, v = synth.draw_qkv(gen, nq, shape)
        pr.query(sid, q, name="query A nq=%d" % nq)
        pr.query(sid, q, k, v, name="query B nq=%d" % nq)
        for S in (1, 2, 7):
            pr.query(sid, q, n_splits=S, name="query A nq=%d S=%d" % (nq, S))
            pr.query(sid, q, k, v, n_splits=S, name="query B nq=%d S=%d" % (nq, S))
    torch.cuda.synchronize()
    assert torch.equal(before, pr.pool.kv_mem)


def test_bf16_first_tokens_short_context():
    """Short contexts (n < 16), where the bf16 rounding of the softmax weights weighs most, and
    the very first token of an empty session (output = its own value, to fp32 rounding)."""
    shape = synth.CFG2
    gen = synth.generator(2, stream=2)
    pr = Pair(shape, n_blocks=16, kv_fill=0xFF)
    sid = pr.create()
    q, k, v = synth.draw_qkv(gen, 1, shape)
    out, lse = pr.append(sid, q, k, v, name="first token")
    G = shape.group
    torch.cuda.synchronize()
    expect = v.float().repeat_interleave(G, dim=1)
    # one key: the weight is exp2(fma(s, c, -round(s*c))), which is 1 up to one rounding of s*c
    assert torch.allclose(out.cpu(), expect, rtol=1e-6, atol=0)
    for L in [1, 2, 3, 5]:
        q, k, v = synth.draw_qkv(gen, L, shape)
        pr.append(sid, q, k, v, name="short append L=%d" % L)
    q, k, v = synth.draw_qkv(gen, 3, shape)
    pr.query(sid, q, name="short query A")
    pr.query(sid, q, k, v, name="short query B")
    pr.check_cache(sid)


def test_bf16_output_dtype_bf16_and_no_lse():
    shape = synth.CFG2
    gen = synth.generator(2, stream=3)
    pr = Pair(shape, n_blocks=64)
    sid = pr.create()
    q, k, v = synth.draw_qkv(gen, 300, shape)
    out, lse = pr.append(sid, q, k, v, out_dtype="bf16", want_lse=False)
    assert out.dtype == torch.bfloat16 and lse is None
    q, k, v = synth.draw_qkv(gen, 32, shape)
    pr.query(sid, q, out_dtype="bf16", n_splits=4, name="bf16 out, split")
    pr.query(sid, q, out_dtype="bf16", n_splits=1, name="bf16 out, direct")


@pytest.mark.parametrize("shape", [synth.Shape("bf16", 8, 8, 64), synth.Shape("bf16", 12, 4, 128),
                                   synth.Shape("f32", 8, 2, 128), synth.Shape("bf16", 64, 8, 128),
                                   synth.Shape("bf16", 8, 8, 128), synth.Shape("bf16", 32, 2, 128),
                                   synth.Shape("bf16", 32, 1, 128)])
def test_other_shapes(shape):
    """fp32 goes through the fp32 kernel; bf16 with G = 32, 16, 8, 3 and 1 through the MFMA kernel
    (a wave's 32 rows are then one token's heads, two tokens, four tokens, ten tokens and two thirds
    of another, 32 tokens), head_dim 64 included."""
    gen = synth.generator(9, stream=shape.n_q_heads)
    pr = Pair(shape, n_blocks=64)
    sid = pr.create()
    for L in [70, 3, 130]:
        q, k, v = synth.draw_qkv(gen, L, shape)
        pr.append(sid, q, k, v, name="append L=%d" % L)
    pr.check_cache(sid)
    q, k, v = synth.draw_qkv(gen, 9, shape)
    pr.query(sid, q, name="query A")
    pr.query(sid, q, k, v, n_splits=2, name="query B")


@pytest.mark.parametrize("hq,hkv,d", [(28, 4, 128), (12, 4, 128), (40, 8, 128), (6, 1, 128),
                                      (32, 8, 64), (14, 2, 64), (8, 8, 64), (16, 1, 64),
                                      (48, 1, 128), (71, 1, 64), (128, 1, 128)])
def test_group_sizes_and_head_dim_64_on_the_matrix_pipe(hq, hkv, d):
    """G = 7, 3, 5 and 6 on the matrix-pipe kernels: a tile holds floor(rows / G) tokens, its last rows
    idle, and a token's heads can lie in two waves.  head_dim 64 (G = 4, 7, 1, 16) on the same kernels:
    half of every K row and of the V^T dims of a tile.  Multi-query shapes with 48, 71 and 128 heads on one
    KV head: a token then fills most of a tile, or two waves and more.  Appends over several row tiles, queries that
    take the 64-, 128- and 256-row instances in both modes and with several split counts, a sliding
    window, a batched step and a question batch."""
    shape = synth.Shape("bf16", hq, hkv, d)
    G = hq // hkv
    gen = synth.generator(9, stream=100 + hq)
    pr = Pair(shape, n_blocks=200, max_sessions=3, max_batch_tokens=1024, kv_fill=0xFF)
    sid = pr.create()
    for L in [300, 1, 37, 150]:
        q, k, v = synth.draw_qkv(gen, L, shape)
        pr.append(sid, q, k, v, name="append L=%d" % L)
        assert pr.pool.sk_pool_last_launch()["kernel_variant"] != 0
    pr.check_cache(sid)
    for rows in (64, 128, 256, 300):
        nq = max(1, rows // G)
        q, k, v = synth.draw_qkv(gen, nq, shape)
        pr.query(sid, q, name="query A nq=%d" % nq)
        assert pr.pool.sk_pool_last_launch()["kernel_variant"] != 0
        for S in (1, 3):
            pr.query(sid, q, k, v, n_splits=S, name="query B nq=%d S=%d" % (nq, S))
    pr.freeze(sid, 33)
    pr.evict(sid, 101)
    q, k, v = synth.draw_qkv(gen, 21, shape)
    pr.query(sid, q, name="query A behind a hole")
    pr.append(sid, q, k, v, name="append behind a hole")
    pr.check_cache(sid)
    # batched step: an append on a second session and a query on the first
    other = pr.create()
    counts = [90, 17]
    cu = np.concatenate([[0], np.cumsum(counts)]).astype(np.int32)
    q, k, v = synth.draw_qkv(gen, int(cu[-1]), shape)
    out, lse = pr.pool.sk_batch_step([other, sid], [sk.SK_OP_APPEND, sk.SK_OP_QUERY_B], cu, dev(q), dev(k), dev(v))
    qr, kr, vr = synth.to_raw(q), synth.to_raw(k), synth.to_raw(v)
    ro0, rl0 = pr.oracles[other].append(qr[:90], kr[:90], vr[:90])
    ro1, rl1 = pr.oracles[sid].query(qr[90:], kr[90:], vr[90:])
    compare("batch step", out, lse, np.concatenate([ro0, ro1]), np.concatenate([rl0, rl1]), shape.dtype)
    pr.check_cache(other)
    # question batch
    P_, NQ, Sfx = 16, 5, 8
    qp, kp, vp = synth.draw_qkv(gen, P_, shape)
    qs, ks, vs = [t.reshape(NQ, Sfx, t.shape[1], d) for t in synth.draw_qkv(gen, NQ * Sfx, shape)]
    op, lp, os_, ls = pr.pool.sk_session_query_shared_prefix(sid, dev(qp), dev(kp), dev(vp), dev(qs), dev(ks), dev(vs))
    rop, rlp, ros, rls = pr.oracles[sid].query_shared_prefix(synth.to_raw(qp), synth.to_raw(kp), synth.to_raw(vp),
                                                             synth.to_raw(qs), synth.to_raw(ks), synth.to_raw(vs))
    compare("question batch, prefix", op, lp, rop, rlp, shape.dtype)
    compare("question batch, suffixes", os_.reshape(NQ * Sfx, hq, d), ls.reshape(NQ * Sfx, hq),
            ros.reshape(NQ * Sfx, hq, d), rls.reshape(NQ * Sfx, hq), shape.dtype)


def test_large_logits_and_needle():
    """Queries scaled by 8 (scores of magnitude ~8 sigma) prove the max subtraction; a planted key
    aligned with the query at several positions (first, last, block and split boundaries) must
    return that key's value: exact retrieval from mid-context (the paper's Q6 idea, Sec. 4.3)."""
    shape = synth.CFG2
    gen = synth.generator(2, stream=4)
    n = 2048
    for pos in [0, 15, 16, 511, 512, 1023, 1024, n - 1]:
        pr = Pair(shape, n_blocks=n // 16 + 4)
        sid = pr.create()
        q, k, v = synth.draw_qkv(gen, n, shape)
        qq, _, _ = synth.draw_qkv(gen, 4, shape, scale=8.0)
        # plant: key at `pos` of KV head 2 is 4x query row (token 1, head 9); head 9 reads KV head 2
        k[pos, 2] = (4.0 * qq[1, 9].float()).to(torch.bfloat16)
        pr.append(sid, q[:1024], k[:1024], v[:1024], check=False)
        pr.append(sid, q[1024:], k[1024:], v[1024:], check=False)
        out, _ = pr.query(sid, qq, n_splits=4, name="needle pos=%d" % pos)
        torch.cuda.synchronize()
        got = out[1, 9].cpu()
        assert torch.allclose(got, v[pos, 2].float(), atol=1e-2), "needle at %d not retrieved" % pos


@pytest.mark.parametrize("hq,hkv,d,env", [(32, 8, 128, None), (32, 8, 64, None), (28, 4, 128, None), (8, 8, 128, None),
                                          (32, 1, 128, None), (14, 2, 64, None), (32, 8, 128, {"SK_SMALL_DISTRUST": "1"}),
                                          (28, 4, 128, {"SK_SMALL_DISTRUST": "1"})])
def test_calls_of_at_most_32_rows(hq, hkv, d, env):
    """The kernel for at most 32 query rows per KV head: empty caches, cached lengths around its tiles, its
    parts and its workgroups' shares, the call's own tokens in a part of their own or in the last one, appends
    whose commit runs in the same launch (starting inside a 16-token group and across two), the merge by the
    last workgroup, the combine kernel behind it, and the recomputation it falls back to."""
    shape = synth.Shape("bf16", hq, hkv, d)
    G = hq // hkv
    gen = synth.generator(2, stream=600 + hq + d)
    lengths = [0, 1, 15, 31, 33, 96, 97, 128, 129, 500, 1100] if env is None else [0, 97, 500]
    for n in lengths:
        pr = Pair(shape, n_blocks=n // 16 + 12, max_sessions=1, kv_fill=0xFF, env=env)
        sid = pr.create()
        if n:
            q, k, v = synth.draw_qkv(gen, n, shape)
            pr.pool.sk_session_append(sid, None, dev(k), dev(v))
            pr.oracles[sid].K, pr.oracles[sid].V = synth.to_raw(k), synth.to_raw(v)
        for nq in sorted({1, max(1, 16 // G), 32 // G}):
            q, k, v = synth.draw_qkv(gen, nq, shape)
            for S in (0, 1, 3):
                if n:
                    pr.query(sid, q, n_splits=S, name="query A n=%d nq=%d S=%d" % (n, nq, S))
                    assert pr.pool.sk_pool_last_launch()["kernel_variant"] == 5
                pr.query(sid, q, k, v, n_splits=S, name="query B n=%d nq=%d S=%d" % (n, nq, S))
            pr.query(sid, q, k, v, name="bf16 results", out_dtype="bf16")
            pr.append(sid, q, k, v, name="append n=%d L=%d" % (n, nq))
            assert pr.pool.sk_pool_last_launch()["kernel_variant"] == 5
            pr.check_cache(sid)
        if n >= 97:
            pr.freeze(sid, 20)
            pr.evict(sid, 45)
            q, k, v = synth.draw_qkv(gen, 32 // G, shape)
            pr.query(sid, q, k, v, name="query B behind a hole")
            pr.append(sid, q, k, v, name="append behind a hole")


@pytest.mark.parametrize("block", [64, 256])
@pytest.mark.parametrize("shape", [synth.Shape("bf16", 32, 8, 128), synth.Shape("bf16", 14, 2, 64), synth.Shape("f32", 8, 2, 128)])
def test_one_launch_calls_with_larger_blocks_and_many_parts(shape, block):
    """The kernels that read a call's own tokens in place, with blocks of several 16-token groups: commits that start
    inside a group, at a block's end and across it, evicted tokens, and parts for one round of the merge and for more,
    up to those that one workgroup still merges (64; in fp32, with these rows, 48: the 59 of n_splits = 60 are merged in bf16 alone)."""
    gen = synth.generator(2, stream=1300 + block + shape.head_dim)
    pr = Pair(shape, block_tokens=block, n_blocks=4200 // block + 6, max_sessions=1, max_batch_tokens=4096, kv_fill=0xFF)
    sid = pr.create()
    ref = pr.oracles[sid]
    G = shape.n_q_heads // shape.n_kv_heads
    for grow in (block - 3, 1000, 2700 - block):
        _, k, v = synth.draw_qkv(gen, grow, shape)
        pr.pool.sk_session_append(sid, None, dev(k), dev(v))
        ref.K, ref.V = np.concatenate([ref.K, synth.to_raw(k)]), np.concatenate([ref.V, synth.to_raw(v)])
        for T in (1, 32 // G, 7):
            if T * G <= 32 or shape.dtype == "f32":
                q, k, v = synth.draw_qkv(gen, T, shape)
                launches = pr.pool.sk_pool_get_stats()["launches"]
                pr.append(sid, q, k, v, name="append %d behind %d" % (T, len(ref.K)))
                geo = pr.pool.sk_pool_last_launch()
                assert pr.pool.sk_pool_get_stats()["launches"] == launches + (2 if geo["n_splits"] > 1 and not geo["fused_merge"] else 1)
                pr.query(sid, q, k, v, name="query B")
    pr.check_cache(sid)
    n = len(ref.K)
    q, k, v = synth.draw_qkv(gen, 1, shape)
    for S in (33, 60):
        pr.query(sid, q, n_splits=S, name="S=%d" % S)
        geo = pr.pool.sk_pool_last_launch()
        assert geo["fused_merge"] == (S == 33 or shape.dtype == "bf16") and geo["n_splits"] == -(-n // (128 if S == 33 else 64)), geo
    pr.freeze(sid, 20)
    pr.evict(sid, block + 9)
    pr.append(sid, q, k, v, name="append behind a hole")
    pr.query(sid, q, k, v, n_splits=60, name="query B behind a hole")
    pr.check_cache(sid)


@pytest.mark.parametrize("hq,hkv,d,most,parts", [(4, 1, 128, 8192, 32), (4, 4, 64, 16384, 32), (12, 12, 128, 4096, 16), (10, 10, 64, 8192, 16)])
def test_short_calls_where_the_kv_heads_do_not_fill_the_xcds(hq, hkv, d, most, parts):
    """With KV heads that are no multiple of 8 the parts are merged in the launch (and cut for the CUs of one XCD) up to
    `most` cached tokens, behind that by the combine kernel; 40 parts that only a caller's n_splits asks for, and the
    64 parts that the combine kernel is given at most, among them."""
    shape = synth.Shape("bf16", hq, hkv, d)
    gen = synth.generator(2, stream=1200 + hq + d)
    pr = Pair(shape, n_blocks=(most + 40) // 16 + 300, max_sessions=1, max_batch_tokens=4096)
    sid = pr.create()
    ref = pr.oracles[sid]
    k, v = [], []

    def grow(n):
        while ref.K.shape[0] < n:
            _, k, v = synth.draw_qkv(gen, min(4096, n - ref.K.shape[0]), shape)
            pr.pool.sk_session_append(sid, None, dev(k), dev(v))
            ref.K, ref.V = np.concatenate([ref.K, synth.to_raw(k)]), np.concatenate([ref.V, synth.to_raw(v)])

    for n, merged in ((most, True), (most + 1, False), (most + 4000, False)):
        grow(n)
        for nq, S in ((1, 0), (2, 0), (2, 40)):
            q, k, v = synth.draw_qkv(gen, nq, shape)
            pr.query(sid, q, n_splits=S, name="query A n=%d nq=%d S=%d" % (n, nq, S))
            geo = pr.pool.sk_pool_last_launch()
            assert geo["kernel_variant"] == 5 and geo["fused_merge"] == (merged and (S == 0 or d == 64 or nq * hq // hkv <= 8))
            if S == 0:
                assert geo["n_splits"] == parts if merged else geo["n_splits"] <= 64
            pr.query(sid, q, k, v, n_splits=S, name="query B n=%d nq=%d S=%d" % (n, nq, S))
        q, k, v = synth.draw_qkv(gen, 1, shape)
        pr.append(sid, q, k, v, name="append n=%d" % n)
        pr.pool.sk_session_truncate(sid, n)
        ref.truncate(n)


@pytest.mark.parametrize("hq,hkv,d,env", [(4, 4, 64, None), (8, 2, 128, None), (16, 1, 64, None), (10, 2, 128, None),
                                          (8, 2, 128, {"SK_SMALL_DISTRUST": "1"})])
def test_fp32_kernel(hq, hkv, d, env):
    """The fp32 kernel: cached lengths around its 16-key tiles and 64-key parts, row tiles with idle rows (5 heads
    per KV head), the call's own tokens behind a padded last tile, commits in the attention launch and (more than
    128 tokens) in front of it, evicted tokens, every merge."""
    shape = synth.Shape("f32", hq, hkv, d)
    gen = synth.generator(1, stream=700 + hq + d)
    for n in ([0, 1, 15, 16, 17, 63, 65, 200, 1300] if env is None else [65, 200]):
        pr = Pair(shape, n_blocks=n // 16 + 40, max_sessions=1, kv_fill=0xFF, env=env)
        sid = pr.create()
        if n:
            q, k, v = synth.draw_qkv(gen, n, shape)
            pr.pool.sk_session_append(sid, None, dev(k), dev(v))
            pr.oracles[sid].K, pr.oracles[sid].V = synth.to_raw(k), synth.to_raw(v)
        for nq in (1, 3, 20):
            q, k, v = synth.draw_qkv(gen, nq, shape)
            for S in (0, 1, 3):
                if n:
                    pr.query(sid, q, n_splits=S, name="query A n=%d nq=%d S=%d" % (n, nq, S))
                pr.query(sid, q, k, v, n_splits=S, name="query B n=%d nq=%d S=%d" % (n, nq, S))
        if n >= 65:
            pr.freeze(sid, 20)
            pr.evict(sid, 33)
        for L in (5, 64, 150):
            q, k, v = synth.draw_qkv(gen, L, shape)
            pr.append(sid, q, k, v, name="append n=%d L=%d" % (n, L))
        k, v = pr.pool.sk_session_gather(sid)
        Kc, Vc = pr.oracles[sid].cache()
        np.testing.assert_array_equal(synth.to_raw(k.cpu()), Kc)
        np.testing.assert_array_equal(synth.to_raw(v.cpu()), Vc)


@pytest.mark.parametrize("hq,hkv,d", [(32, 8, 128), (32, 8, 64), (4, 4, 128), (4, 4, 64), (28, 4, 128), (71, 1, 64)])
def test_own_tokens_of_a_query_staged_by_the_attention_kernel(hq, hkv, d):
    """Queries of one row tile per KV head stage their own K/V (up to 64 tokens) in the workgroup of the own part: token
    counts around 16-token groups, at the row tiles' edges, and around the two limits behind which a launch in front
    stages them; empty and short caches, and a cache long enough for the eight-wave 128-row instance; what an
    earlier call left behind the last token (NaN) never counts."""
    shape = synth.Shape("bf16", hq, hkv, d)
    G = hq // hkv
    gen = synth.generator(2, stream=900 + hq + d)
    counts = sorted({c for c in (1, 15, 16, 17, 33, 48, 63, 64, 65, 32 // G + 1, 64 // G, 64 // G + 1, 128 // G, 128 // G + 1,
                                 256 // G, 256 // G + 1) if c > 0 and 32 < c * G <= 300})
    for n, env in ((0, None), (33, None), (700, None), (700, LONG_CACHE_PATHS)):
        pr = Pair(shape, n_blocks=n // 16 + 12, max_sessions=1, kv_fill=0xFF, env=env)
        sid = pr.create()
        if n:
            q, k, v = synth.draw_qkv(gen, n, shape)
            pr.pool.sk_session_append(sid, None, dev(k), dev(v))
            pr.oracles[sid].K, pr.oracles[sid].V = synth.to_raw(k), synth.to_raw(v)
        for nq in counts:
            q, k, v = synth.draw_qkv(gen, 64, shape)
            pr.pool.sk_session_query(sid, dev(q), dev(k), dev(v * float("nan")))
            q, k, v = synth.draw_qkv(gen, nq, shape)
            pr.query(sid, q, k, v, n_splits=0 if nq % 2 else 3, name="query B n=%d nq=%d" % (n, nq))
        pr.query(sid, q, k, v, name="bf16 results", out_dtype="bf16")


@pytest.mark.parametrize("hd", [128, 64])
@pytest.mark.parametrize("env", [None, LONG_CACHE_PATHS])
def test_scores_that_grow_along_the_cache(hd, env):
    """The kernels weigh a tile against the maximum they have and look for a new one only when the sum of
    the weights says so: keys whose size grows in steps (by a little, so that weights stay just below the
    limit, and by much, so that they overflow to infinity first), and one that falls again, for every
    kernel instance, with masked tiles among them."""
    shape = synth.Shape("bf16", 32, 8, hd)
    gen = synth.generator(2, stream=400 + hd)
    n = 900
    pr = Pair(shape, n_blocks=n // 16 + 30, max_sessions=2, max_batch_tokens=1024, env=env)
    sid = pr.create()
    q, k, v = synth.draw_qkv(gen, n, shape)
    grow = torch.ones(n)
    for at, f in ((64, 1.5), (130, 1.2), (200, 3.0), (300, 0.2), (500, 12.0), (515, 60.0), (600, 0.5), (700, 2.5)):
        grow[at:] *= f
    k = (k.float() * grow[:, None, None]).to(torch.bfloat16)
    for a, b in ((0, 5), (5, 400), (400, n)):
        pr.append(sid, q[a:b], k[a:b], v[a:b], name="append %d:%d" % (a, b))
    for nq in (1, 16, 32, 60):
        for S in (0, 1, 3):
            pr.query(sid, q[:nq], n_splits=S, name="query A nq=%d S=%d" % (nq, S))
            pr.query(sid, q[:nq], k[-nq:], v[-nq:], n_splits=S, name="query B nq=%d S=%d" % (nq, S))


@pytest.mark.parametrize("hq,hkv,d", [(4, 4, 64), (10, 2, 128)])
def test_fp32_negative_softmax_scale(hq, hkv, d):
    """softmax_scale may be negative: the smallest product then has the largest weight.  Scores of a few hundred (a
    scale of -8), so that a weight taken against the wrong end of a row overflows; tiles that end inside a 16-key group,
    causal limits and evicted tokens, so that masked keys are among them.  Scores of that size cost digits: a
    product of d terms carries 2^-24 * |score| * log2(e) of absolute error into the exponent, here about 1e-4, which is
    a weight's relative error, and with it the output's and the log-sum-exp's."""
    shape = synth.Shape("f32", hq, hkv, d)
    gen = synth.generator(1, stream=40 + hq)
    pr = Pair(shape, n_blocks=80, max_sessions=1, kv_fill=0xFF, softmax_scale=-8.0)
    sid = pr.create()

    def close(name, out, lse, ro, rl):
        og, lg = out.double().cpu().numpy(), lse.double().cpu().numpy()
        assert np.isfinite(og).all() and np.isfinite(lg).all(), name
        assert np.abs(og - ro).max() <= 2e-3 and np.abs(lg - rl).max() <= 2e-3, name

    ref = pr.oracles[sid]
    for n in (1, 40, 205, 3, 400):
        q, k, v = synth.draw_qkv(gen, n, shape)
        raw = [synth.to_raw(t) for t in (q, k, v)]
        close("append %d" % n, *pr.pool.sk_session_append(sid, dev(q), dev(k), dev(v)), *ref.append(*raw))
    for evicted in (0, 33):
        if evicted:
            pr.freeze(sid, 20)
            pr.evict(sid, evicted)
        for nq in (1, 20):
            q, k, v = synth.draw_qkv(gen, nq, shape)
            raw = [synth.to_raw(t) for t in (q, k, v)]
            for S in (0, 1, 3):
                close("query A", *pr.pool.sk_session_query(sid, dev(q), n_splits=S), *ref.query(raw[0]))
                close("query B", *pr.pool.sk_session_query(sid, dev(q), dev(k), dev(v), n_splits=S), *ref.query(*raw))


@pytest.mark.parametrize("n", [1, 5, 16, 17, 31, 70])
def test_fp32_infinite_value_of_the_last_token(n):
    """An infinite value reaches the output dimension it stands in, and nothing else: also from the last cached token
    and the last token of the call, whose tile is not full."""
    shape = synth.Shape("f32", 4, 2, 64)
    gen = synth.generator(1, stream=60 + n)
    inf = float("inf")

    def check(name, got, ref, tokens, lse, rl):
        """ref, rl: the oracle's, with a zero in place of the infinities; `tokens`: the rows"""
        got = got.double().cpu().numpy()
        for head, dim in ((0, 3), (1, 40)):
            for t in tokens:
                assert (got[t, 2 * head:2 * head + 2, dim] == inf).all(), name
            got[:, 2 * head:2 * head + 2, dim] = 0.0
            ref[:, 2 * head:2 * head + 2, dim] = 0.0
        assert np.abs(got - ref).max() <= 1e-5 and np.abs(lse.double().cpu().numpy() - rl).max() <= 2e-5, name

    def planted(v):
        w = v.clone()
        w[-1, 0, 3] = inf; w[-1, 1, 40] = inf
        return w

    for own in (False, True):
        pr = Pair(shape, n_blocks=20, max_sessions=1, kv_fill=0xFF)
        sid = pr.create()
        ref = pr.oracles[sid]
        q, k, v = synth.draw_qkv(gen, n, shape)
        v[-1, 0, 3] = 0.0; v[-1, 1, 40] = 0.0
        pr.pool.sk_session_append(sid, None, dev(k), dev(v if own else planted(v)))
        ref.K, ref.V = synth.to_raw(k), synth.to_raw(v)
        q, k, v = synth.draw_qkv(gen, 2, shape)
        for S in (0, 1):
            if own:                                  # one token of its own, which is the last
                k1, v1 = k[:1], v[:1].clone()
                v1[-1, 0, 3] = 0.0; v1[-1, 1, 40] = 0.0
                out, lse = pr.pool.sk_session_query(sid, dev(q[:1]), dev(k1), dev(planted(v1)), n_splits=S)
                ro, rl = ref.query(synth.to_raw(q[:1]), synth.to_raw(k1), synth.to_raw(v1))
                check("own", out, ro, [0], lse, rl)
            else:
                out, lse = pr.pool.sk_session_query(sid, dev(q), n_splits=S)
                ro, rl = ref.query(synth.to_raw(q))
                check("cached", out, ro, range(2), lse, rl)


@pytest.mark.parametrize("hq,hkv,d", [(32, 8, 128), (14, 2, 64)])
@pytest.mark.parametrize("n", [1, 15, 17, 47, 130, 777])
def test_infinite_value_of_a_token_committed_in_the_attention_launch(hq, hkv, d, n):
    """A short append attends to its tokens where the caller has them while the same launch commits them into the
    16-token group in which the cached ones end: what stands behind the cached tokens there never counts, an infinite value
    neither, whenever the commit writes it."""
    shape = synth.Shape("bf16", hq, hkv, d)
    gen = synth.generator(2, stream=1000 + n + d)
    inf = float("inf")
    pr = Pair(shape, n_blocks=n // 16 + 8, max_sessions=1)
    sid = pr.create()
    q, k, v = synth.draw_qkv(gen, n, shape)
    pr.pool.sk_session_append(sid, None, dev(k), dev(v))
    ref = pr.oracles[sid]
    ref.K, ref.V = synth.to_raw(k), synth.to_raw(v)
    q, k, v = synth.draw_qkv(gen, 1, shape)
    v[-1, 0, 3] = 0.0; v[-1, hkv - 1, 40] = 0.0
    ro, rl = ref.query(synth.to_raw(q), synth.to_raw(k), synth.to_raw(v))
    v[-1, 0, 3] = inf; v[-1, hkv - 1, 40] = inf
    qd, kd, vd, G = dev(q), dev(k), dev(v), hq // hkv
    clean = torch.zeros_like(vd)
    for rep in range(8):                       # (the group's free slots hold zeros at first, then what was there before)
        out, lse = pr.pool.sk_session_append(sid, qd, kd, vd)
        pr.pool.sk_session_truncate(sid, n)
        for head, dim in ((0, 3), (hkv - 1, 40)):
            rows = slice(head * G, (head + 1) * G)
            assert bool((out[:, rows, dim] == inf).all()), "pass %d" % rep
            out[:, rows, dim] = 0.0; ro[:, rows, dim] = 0.0
        compare("pass %d" % rep, out, lse, ro, rl, shape.dtype)
        if rep % 2:                            # zeros again
            pr.pool.sk_session_append(sid, None, kd, clean)
            pr.pool.sk_session_truncate(sid, n)


@pytest.mark.parametrize("shape,tokens", [(synth.Shape("bf16", 8, 8, 128), (1, 20, 60)), (synth.Shape("bf16", 4, 4, 64), (3, 32, 70)),
                                          (synth.Shape("bf16", 32, 8, 128), (5, 16)), (synth.Shape("f32", 4, 4, 64), (3, 60, 150))])
@pytest.mark.parametrize("n", [0, 40, 1100])
def test_results_over_the_calls_own_keys_and_values(shape, tokens, n):
    """The buffers of a call's own k and v may be given for its results too: the keys and values count as they were when
    the call was made, and an append commits them so.  fp32 results over k and v that lie one behind the other, results
    of the pool's type exactly over v, and the log-sum-exp over k."""
    gen = synth.generator(2, stream=1100 + n + shape.n_q_heads)
    pr = Pair(shape, n_blocks=n // 16 + 60, max_sessions=1)
    sid = pr.create()
    ref = pr.oracles[sid]
    if n:
        q, k, v = synth.draw_qkv(gen, n, shape)
        pr.pool.sk_session_append(sid, None, dev(k), dev(v))
        ref.K, ref.V = synth.to_raw(k), synth.to_raw(v)
    el = 2 if shape.dtype == "bf16" else 4
    rows, d = shape.n_q_heads, shape.head_dim
    for T in tokens:
        for call in (pr.pool.sk_session_query, pr.pool.sk_session_append):
            for how in ("f32 over both", "over v", "lse over k"):
                q, k, v = synth.draw_qkv(gen, T, shape)
                if call == pr.pool.sk_session_query:
                    ro, rl = ref.query(synth.to_raw(q), synth.to_raw(k), synth.to_raw(v))
                else:
                    ro, rl = ref.append(synth.to_raw(q), synth.to_raw(k), synth.to_raw(v))
                own = k.numel() * el
                buf = torch.empty(max(2 * own, own + T * rows * d * 4), dtype=torch.uint8, device="cuda")
                kd, vd = (buf[a:a + own].view(k.dtype).view(k.shape) for a in (0, own))
                kd.copy_(dev(k)); vd.copy_(dev(v))
                out_dtype = shape.dtype if how == "over v" else "f32"
                out = torch.empty((T, rows, d), dtype=torch.float32, device="cuda")
                lse = torch.empty((T, rows), dtype=torch.float32, device="cuda")
                if how == "f32 over both":
                    out = buf[:T * rows * d * 4].view(torch.float32).view(T, rows, d)
                elif how == "over v":
                    out = buf[own:own + T * rows * d * el].view(k.dtype).view(T, rows, d)
                else:
                    lse = buf[:T * rows * 4].view(torch.float32).view(T, rows)
                call(sid, dev(q), kd, vd, out=out, lse=lse, out_dtype=out_dtype)
                compare("%s T=%d %s" % (call.__name__, T, how), out, lse, ro, rl, shape.dtype, out_dtype == "bf16")
    pr.check_cache(sid)


@pytest.mark.parametrize("shape,n,parts", [(synth.Shape("bf16", 32, 8, 128), 2592, 21), (synth.Shape("bf16", 14, 2, 64), 1184, 10),
                                           (synth.Shape("f32", 4, 2, 64), 80, 2)])
def test_infinite_value_in_the_last_part_of_a_merged_call(shape, n, parts):
    """The workgroup that merges reads sixteen parts at a time: an infinite value of the last part reaches the output
    dimension it stands in and is not met by a weight of 0 where the sixteen are not full."""
    gen = synth.generator(2, stream=60 + n)
    inf = float("inf")
    pr = Pair(shape, n_blocks=n // 16 + 8, max_sessions=1)
    sid = pr.create()
    ref = pr.oracles[sid]
    q, k, v = synth.draw_qkv(gen, n, shape)
    v[-1, 0, 3] = 0.0
    ref.K, ref.V = synth.to_raw(k), synth.to_raw(v)
    v[-1, 0, 3] = inf
    pr.pool.sk_session_append(sid, None, dev(k), dev(v))
    q, _, _ = synth.draw_qkv(gen, 2, shape)
    out, lse = pr.pool.sk_session_query(sid, dev(q))
    geo = pr.pool.sk_pool_last_launch()
    assert geo["fused_merge"] == 1 and geo["n_splits"] == parts and parts % 8
    G = shape.n_q_heads // shape.n_kv_heads
    assert bool((out[:, :G, 3] == inf).all())
    ro, rl = ref.query(synth.to_raw(q))
    out[:, :G, 3] = 0.0; ro[:, :G, 3] = 0.0
    compare("last part", out, lse, ro, rl, shape.dtype)


@pytest.mark.parametrize("scale", [0.05, 0.2])
def test_custom_softmax_scale(scale):
    """Eq. 1's 1/sqrt(d_k) is the default, not the only scale: a pool created with softmax_scale set
    (0.05 flattens the weights, 0.2 sharpens them well beyond 1/sqrt(128) = 0.088) against an oracle
    given the same number, through every entry point: appends (several row tiles, split merge),
    cache-only and own-K/V queries with several split counts, a ragged multi-session step and a
    shared-prefix question batch; fp32 pool once as well."""
    import oracle
    import paper_2605_13784_amd as sk
    shape = synth.CFG2
    gen = synth.generator(2, stream=300 + int(scale * 100))
    pr = Pair(shape, block_tokens=16, n_blocks=400, max_sessions=3, max_batch_tokens=1024, softmax_scale=scale)
    a, b = pr.create(), pr.create()
    for sid, Ls in ((a, [300, 700, 41]), (b, [90, 1])):
        for L in Ls:
            q, k, v = synth.draw_qkv(gen, L, shape)
            pr.append(sid, q, k, v, name="scale %.2f append %d" % (scale, L))
    for nq in (32, 5):
        q, k, v = synth.draw_qkv(gen, nq, shape)
        for S in (0, 1, 5):
            pr.query(a, q, n_splits=S, name="scale %.2f query A nq=%d S=%d" % (scale, nq, S))
            pr.query(a, q, k, v, n_splits=S, name="scale %.2f query B nq=%d S=%d" % (scale, nq, S))
    # ragged step: append on b, own-K/V query on a
    counts = [130, 20]
    cu = np.concatenate([[0], np.cumsum(counts)]).astype(np.int32)
    q, k, v = synth.draw_qkv(gen, int(cu[-1]), shape)
    out, lse = pr.pool.sk_batch_step([b, a], [sk.SK_OP_APPEND, sk.SK_OP_QUERY_B], cu, dev(q), dev(k), dev(v))
    qr, kr, vr = synth.to_raw(q), synth.to_raw(k), synth.to_raw(v)
    ro, rl = pr.oracles[b].append(qr[:130], kr[:130], vr[:130])
    compare("scale %.2f step append" % scale, out[:130], lse[:130], ro, rl, shape.dtype)
    ro, rl = pr.oracles[a].query(qr[130:], kr[130:], vr[130:])
    compare("scale %.2f step query" % scale, out[130:], lse[130:], ro, rl, shape.dtype)
    pr.check_cache(b)
    # question batch on a
    P, NQ, Sfx = 16, 6, 8
    qp, kp, vp = synth.draw_qkv(gen, P, shape)
    qs, ks, vs = synth.draw_qkv(gen, NQ * Sfx, shape)
    r4 = lambda t: t.reshape(NQ, Sfx, t.shape[1], shape.head_dim)
    op, lp, os_, ls = pr.pool.sk_session_query_shared_prefix(a, dev(qp), dev(kp), dev(vp), dev(r4(qs)), dev(r4(ks)), dev(r4(vs)))
    rop, rlp, ros, rls = pr.oracles[a].query_shared_prefix(synth.to_raw(qp), synth.to_raw(kp), synth.to_raw(vp),
                                                           synth.to_raw(r4(qs)), synth.to_raw(r4(ks)), synth.to_raw(r4(vs)))
    compare("scale %.2f prefix" % scale, op, lp, rop, rlp, shape.dtype)
    compare("scale %.2f suffixes" % scale, os_, ls, ros, rls, shape.dtype)
    # the fp32 path takes the scale the same way
    pf = Pair(synth.CFG1, block_tokens=16, n_blocks=40, softmax_scale=scale)
    s = pf.create()
    q, k, v = synth.draw_qkv(gen, 100, synth.CFG1)
    pf.append(s, q, k, v, name="fp32 scale %.2f append" % scale)
    q, k, v = synth.draw_qkv(gen, 9, synth.CFG1)
    pf.query(s, q, n_splits=3, name="fp32 scale %.2f query A" % scale)
    pf.query(s, q, k, v, name="fp32 scale %.2f query B" % scale)


@pytest.mark.parametrize("hq,hkv,d", [(32, 8, 128), (14, 2, 64)])
def test_combine_rounds(hq, hkv, d):
    """The combine kernel asks for 8, 16 or 32 parts at once, by the parts of the launch: both sides of each border, more parts
    than one round and than the 64 whose statistics one wave holds, results in fp32 and bf16."""
    shape = synth.Shape("bf16", hq, hkv, d)
    gen = synth.generator(2, stream=1500 + d)
    nq = 40 // (hq // hkv)
    pr = Pair(shape, n_blocks=72 * 4 + 8, max_sessions=1, max_batch_tokens=4096)
    sid = pr.create()
    for t in range(0, 72 * 64, 1152):
        _, k, v = synth.draw_qkv(gen, 1152, shape)
        pr.append(sid, None, k, v, check=False)
    q, k, v = synth.draw_qkv(gen, nq, shape)
    for S in (72, 65, 64, 33, 32, 31, 17, 16, 9, 8, 7, 2):
        pr.pool.sk_session_truncate(sid, 64 * S)
        pr.oracles[sid].truncate(64 * S)
        for own in (False, True):              # the own part is one more
            pr.query(sid, q, k if own else None, v if own else None, n_splits=S, out_dtype="bf16" if S % 2 else "f32", name="S=%d own=%d" % (S, own))
            geo = pr.pool.sk_pool_last_launch()
            assert geo["n_splits"] == S + own and geo["fused_merge"] == 0, geo


@pytest.mark.parametrize("hq,hkv,frozen", [(32, 8, 5), (14, 2, 300)])
def test_head_dim_64_tiles_of_256_rows(hq, hkv, frozen):
    """The 256-row instance at head_dim 64: cached lengths at the edges of a tile (32 keys), of an iteration (64) and of
    the ring (eight tiles), one and several row tiles with ragged last rows, direct and split results, queries with and without
    their own K/V, evicted tokens in the first and in a middle tile."""
    shape = synth.Shape("bf16", hq, hkv, 64)
    gen = synth.generator(2, stream=1600 + hq)
    G = hq // hkv
    pr = Pair(shape, n_blocks=400, max_sessions=1, max_batch_tokens=1024, kv_fill=0xFF)
    sid = pr.create()
    ref = pr.oracles[sid]
    variants = set()
    for n in (0, 1, 31, 33, 64, 96, 97, 160, 224, 255, 257, 288, 320, 545, 900):
        if n > len(ref.K):
            _, k, v = synth.draw_qkv(gen, n - len(ref.K), shape)
            pr.append(sid, None, k, v, check=False)
        for T in (128 // G + 1, 256 // G, 256 // G + 1) if n in (0, 33, 257, 900) else (256 // G - 3,):
            q, k, v = synth.draw_qkv(gen, T, shape)
            for S in (1, 3):                   # (with a number of parts of the caller's always this instance)
                if n:
                    pr.query(sid, q, n_splits=S, name="A n=%d T=%d S=%d" % (n, T, S))
                    assert pr.pool.sk_pool_last_launch()["kernel_variant"] == 3
                pr.query(sid, q, k, v, n_splits=S, name="B n=%d T=%d S=%d" % (n, T, S))
                assert pr.pool.sk_pool_last_launch()["kernel_variant"] == 3
            pr.append(sid, q, k, v, name="append n=%d T=%d" % (n, T))
            variants.add(pr.pool.sk_pool_last_launch()["kernel_variant"])
            pr.pool.sk_session_truncate(sid, n)
            ref.truncate(n)
    for T in (1024,) * 4 + (40,):              # a long append behind a longer cache, whose results the tests at full size check
        q, k, v = synth.draw_qkv(gen, T, shape)
        pr.append(sid, q, k, v, check=False)
        variants.add(pr.pool.sk_pool_last_launch()["kernel_variant"])
    pr.pool.sk_session_truncate(sid, 900)
    ref.truncate(900)
    assert variants == {1, 3}                  # 128- and 256-row tiles, by the expected end
    pr.freeze(sid, frozen)
    for gone in (20, 40, 200):
        pr.evict(sid, gone)
        q, k, v = synth.draw_qkv(gen, 256 // G, shape)
        pr.query(sid, q, k, v, n_splits=4, name="%d more evicted" % gone)
        pr.query(sid, q, n_splits=1, name="%d more evicted, one part" % gone)
        pr.append(sid, q, k, v, name="append behind a hole")
    pr.check_cache(sid)


@pytest.mark.parametrize("env", [None, {"SK_TARGET_WGS": "256"}])
@pytest.mark.parametrize("hq,hkv,d,n,T", [(28, 4, 128, 0, 502), (12, 4, 128, 100, 500), (4, 1, 64, 0, 600), (16, 1, 128, 0, 900)])
def test_appends_whose_tiles_have_different_numbers_of_parts(hq, hkv, d, n, T, env):
    """Tiles of one part are written directly, the others go through the combine kernel, in one launch: with pieces of at
    least 256 keys for 256 workgroups (env), and with those that are expected to end first."""
    shape = synth.Shape("bf16", hq, hkv, d)
    gen = synth.generator(2, stream=1700 + hq + d)
    pr = Pair(shape, n_blocks=100, max_sessions=1, max_batch_tokens=1024, kv_fill=0xFF, env=env)
    sid = pr.create()
    if n:
        _, k, v = synth.draw_qkv(gen, n, shape)
        pr.append(sid, None, k, v, check=False)
    q, k, v = synth.draw_qkv(gen, T, shape)
    for dt in ("f32", "bf16"):
        pr.append(sid, q, k, v, out_dtype=dt, name="append %d at %d %s" % (T, n, dt))
        geo = pr.pool.sk_pool_last_launch()
        # (with the default plan the first tile of the second and of the last call is one part: it sees no more than 256 keys)
        assert geo["row_tiles"] > 1 and (geo["n_splits"] > 1 or (env is None and (hq, d) not in ((12, 128), (16, 128)))), geo
        pr.pool.sk_session_truncate(sid, n)
        pr.oracles[sid].truncate(n)
    pr.append(sid, q, k, v)
    pr.check_cache(sid)


@pytest.mark.parametrize("shape", [synth.Shape("bf16", 8, 4, 128), synth.Shape("f32", 4, 2, 64)])
def test_long_appends_in_a_row(shape):
    """Appends whose commit lists are too long for the kernel arguments are read from pinned memory by the commit kernel:
    more of them in flight than there are slots, starting inside a group, then one that fits the arguments."""
    gen = synth.generator(2, stream=1800 + shape.head_dim)
    pr = Pair(shape, n_blocks=800, max_sessions=1, max_batch_tokens=2048, kv_fill=0xFF)
    sid = pr.create()
    for L in (1283, 1500, 1300, 1299, 1601, 1290, 2048, 100):
        _, k, v = synth.draw_qkv(gen, L, shape)
        pr.append(sid, None, k, v, check=False)
    pr.check_cache(sid)
    q, k, v = synth.draw_qkv(gen, 5, shape)
    pr.query(sid, q, k, v)


@pytest.mark.parametrize("n,T", [(0, 128), (70, 150), (40, 300)])
def test_head_dim_64_infinite_value_of_a_later_token(n, T):
    """256-row tiles of 128 tokens each (two query heads per KV head): the last token's value is infinite.  A wave computes
    nothing for the 64 keys of an iteration that none of its rows sees, so the rows in front of the iteration that holds
    the infinity give the bits they give with a zero in its place."""
    shape = synth.Shape("bf16", 8, 4, 64)
    gen = synth.generator(2, stream=1900 + T)
    pr = Pair(shape, n_blocks=60, max_sessions=1, max_batch_tokens=1024)
    sid = pr.create()
    if n:
        _, k, v = synth.draw_qkv(gen, n, shape)
        pr.append(sid, None, k, v, check=False)
    q, k, v = synth.draw_qkv(gen, T, shape)
    v[-1, :, 5] = 0.0
    planted = v.clone()
    planted[-1, :, 5] = float("inf")
    def append(v):
        out, lse = pr.pool.sk_session_append(sid, dev(q), dev(k), dev(v))
        variant = pr.pool.sk_pool_last_launch()["kernel_variant"]
        pr.pool.sk_session_truncate(sid, n)
        return out, lse, variant
    def query(v):
        out, lse = pr.pool.sk_session_query(sid, dev(q), dev(k), dev(v), n_splits=1)
        return out, lse, pr.pool.sk_pool_last_launch()["kernel_variant"]
    for call, first in ((append, (n + T - 1) // 64 * 64 - n), (query, (T - 1) // 64 * 64)):      # first token that shares the iteration
        first = first // 16 * 16                                     # a wave holds 16 tokens
        zero, inf = call(v), call(planted)
        assert zero[2] == inf[2] and (call is append or zero[2] == 3)
        assert 0 < first < T and torch.equal(zero[0][:first], inf[0][:first]), call.__name__
        assert torch.equal(zero[1], inf[1]) and not torch.isfinite(inf[0][-1, :, 5]).any(), call.__name__
        ref = pr.oracles[sid].query(synth.to_raw(q), synth.to_raw(k), synth.to_raw(v))
        compare(call.__name__, zero[0], zero[1], *ref, shape.dtype)


@pytest.mark.parametrize("hq,hkv,n,T", [(32, 8, 0, 64), (32, 8, 40, 70), (8, 4, 700, 200)])
def test_head_dim_64_both_tile_heights_round_the_same_weights(hq, hkv, n, T):
    """256- and 128-row tiles take a row's reference maximum from the same 64 keys, so the weights they round to 16 bits are the
    same ones: results equal to fp32 summation error (a reference from 32 keys: 1e-3)."""
    shape = synth.Shape("bf16", hq, hkv, 64)
    gen = synth.generator(2, stream=2000 + T)
    got = []
    q, k, v = synth.draw_qkv(gen, T, shape)
    _, kc, vc = synth.draw_qkv(gen, n, shape)
    for env in (None, {"SK_NO_256": "1"}):
        pr = Pair(shape, n_blocks=80, max_sessions=1, max_batch_tokens=1024, env=env)
        sid = pr.create()
        if n:
            pr.append(sid, None, kc, vc, check=False)
        got.append(pr.pool.sk_session_query(sid, dev(q), dev(k), dev(v), n_splits=1))
        assert pr.pool.sk_pool_last_launch()["kernel_variant"] == (1 if env else 3)
    (a, la), (b, lb) = got
    assert float((a - b).norm() / b.norm()) <= 2e-6 and float((la - lb).abs().max()) <= 2e-5


@pytest.mark.parametrize("hq,hkv,n,T,eight", [(32, 8, 14336, 32, False), (32, 8, 14337, 17, True), (28, 4, 20000, 18, False), (12, 4, 29000, 22, True),
                                              (8, 1, 45000, 16, False), (14, 2, 14800, 18, False), (32, 32, 3585, 66, True), (32, 32, 3584, 128, False)])
def test_eight_waves_from_512_keys_a_workgroup(hq, hkv, n, T, eight):
    """Calls of 65 to 128 rows take the eight-wave instance by the keys of a workgroup, which the number of KV heads decides as
    much as the cached tokens: both sides of the line, single rows against attention in float64."""
    shape = synth.Shape("bf16", hq, hkv, 128)
    gen = torch.Generator(device="cuda").manual_seed(n)
    draw = lambda T, H: torch.randn((T, H, 128), generator=gen, device="cuda").to(torch.bfloat16)
    pool = sk.Pool("bf16", hq, hkv, 128, 16, n // 16 + 8, max_sessions=1)
    sid = pool.sk_session_create()
    K, V = draw(n, hkv), draw(n, hkv)
    for t in range(0, n, 4096):
        pool.sk_session_append(sid, None, K[t:t + 4096], V[t:t + 4096])
    q = draw(T, hq)
    out, lse = pool.sk_session_query(sid, q)
    geo = pool.sk_pool_last_launch()
    assert geo["kernel_variant"] == (4 if eight else 1) and geo["workgroups"] <= 256, geo
    for t, h in ((0, 0), (T - 1, hq - 1), (T // 2, hq // 2)):
        s = (K[:, h // (hq // hkv)].double() @ q[t, h].double()) / 128 ** 0.5
        ref = torch.softmax(s, 0) @ V[:, h // (hq // hkv)].double()
        compare("row %d head %d" % (t, h), out[t, h], lse[t, h], ref.cpu().numpy(), torch.logsumexp(s, 0).cpu().numpy(), shape.dtype)


@pytest.mark.parametrize("hq,hkv,d,T", [(32, 8, 128, 1500), (32, 8, 128, 1750), (32, 8, 128, 2000), (28, 4, 128, 1400), (28, 4, 128, 2300),
                                        (64, 8, 128, 700), (32, 8, 64, 2000)])
def test_one_cached_token_does_not_change_how_an_append_is_cut(hq, hkv, d, T):
    """Row tiles behind an empty session and behind a few tokens are practically the same ones: so are their pieces."""
    gen = torch.Generator(device="cuda").manual_seed(T)
    draw = lambda H, L: torch.randn((L, H, d), generator=gen, device="cuda").to(torch.bfloat16)
    pool = sk.Pool("bf16", hq, hkv, d, 16, T // 16 + 8, max_sessions=1)
    sid = pool.sk_session_create()
    q, k, v = draw(hq, T), draw(hkv, T), draw(hkv, T)
    cut = []
    for n in (0, 1, 16):
        if n:
            pool.sk_session_append(sid, None, k[:n].contiguous(), v[:n].contiguous())
        pool.sk_session_append(sid, q, k, v)
        geo = pool.sk_pool_last_launch()
        cut.append((geo["kernel_variant"], geo["row_tiles"], geo["n_splits"]))
        pool.sk_session_truncate(sid, 0)
    assert cut[0] == cut[1] == cut[2], cut


@pytest.mark.parametrize("heads,n,splits", [(4096, 128, 2), (2048, 576, 9)])
def test_combine_of_parts_beyond_32_bit_offsets(heads, n, splits):
    """With thousands of KV heads the parts of a row lie so far apart that the combine kernel's round does not reach over eight, or
    sixteen, of them within 32-bit offsets: it takes one part at a time, or two rounds of eight.  Against one part and, for some
    heads, attention in float64."""
    T, d = 130, 128
    gen = torch.Generator(device="cuda").manual_seed(heads)
    draw = lambda L: torch.randn((L, heads, d), generator=gen, device="cuda").to(torch.bfloat16)
    pool = sk.Pool("bf16", heads, heads, d, 16, n // 16 + 8, max_sessions=1, max_batch_tokens=256 if splits == 2 else 1280)
    sid = pool.sk_session_create()
    k, v, q = draw(n), draw(n), draw(T)
    for t in range(0, n, 256):
        pool.sk_session_append(sid, None, k[t:t + 256], v[t:t + 256])
    one = pool.sk_session_query(sid, q, n_splits=1)
    assert pool.sk_pool_last_launch()["n_splits"] == 1
    out, lse = pool.sk_session_query(sid, q, n_splits=splits)
    geo = pool.sk_pool_last_launch()
    assert geo["n_splits"] == splits, geo
    step = heads * 256 * d * 4
    assert geo["kernel_variant"] == 3 and (8 if splits == 2 else 16) * step >= 1 << 32
    # two roundings of the weights to 16 bits, against other reference maxima: 2 x 2^-9 of the largest value's share of a row
    assert float((out - one[0]).norm() / one[0].norm()) <= 2.0 ** -8 and float((lse - one[1]).abs().max()) <= 2e-5
    for h in (0, heads // 2 + 1, heads - 1):
        s = (q[:, h].double() @ k[:, h].double().t()) / d ** 0.5
        ref = torch.softmax(s, 1) @ v[:, h].double()
        compare("head %d" % h, out[:, h], lse[:, h], ref.cpu().numpy(), torch.logsumexp(s, 1).cpu().numpy(), "bf16")
