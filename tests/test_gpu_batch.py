"""GPU parity of the batched entry points: the ragged multi-session step and the shared-prefix
question batch, against the fp64 oracle (which defines them as "the same calls one by one")."""
import numpy as np
import pytest
import torch

import oracle
import paper_2605_13784_amd as sk
from workloads import synth
from gpu_common import Pair, compare, dev

pytestmark = pytest.mark.gpu


def _grow(pool, ref, sids, lengths, shape, gen):
    """Round-robin growth in 64-token pieces so that block tables interleave."""
    done = [0] * len(sids)
    while any(d < n for d, n in zip(done, lengths)):
        for i, sid in enumerate(sids):
            L = min(64, lengths[i] - done[i])
            if L <= 0:
                continue
            q, k, v = synth.draw_qkv(gen, L, shape)
            pool.sk_session_append(sid, None, dev(k), dev(v))
            o = ref.sessions[sid]
            o.K = np.concatenate([o.K, synth.to_raw(k)])
            o.V = np.concatenate([o.V, synth.to_raw(v)])
            done[i] += L


def _check_caches(pool, ref, sids):
    for sid in sids:
        k, v = pool.sk_session_gather(sid)
        torch.cuda.synchronize()
        K, V = ref.sessions[sid].cache()
        np.testing.assert_array_equal(synth.to_raw(k.cpu()), K)
        np.testing.assert_array_equal(synth.to_raw(v.cpu()), V)


@pytest.mark.parametrize("shape,n_sessions,lo,hi", [(synth.CFG4, 8, 40, 3000), (synth.CFG1, 5, 10, 400)])
def test_ragged_multi_session_steps(shape, n_sessions, lo, hi):
    """Multi-tenant workload in small: sessions of log-uniform lengths in one pool with 16-token
    blocks handed out in a seeded random order; every step mixes appends on some sessions with
    queries (cache-only and with own K/V) on others."""
    gen = synth.generator(4, stream=n_sessions)
    lengths = synth.loguniform_lengths(gen, n_sessions, lo, hi)
    n_blocks = sum((n + 15) // 16 for n in lengths) + 400
    pool = sk.Pool(shape.dtype, shape.n_q_heads, shape.n_kv_heads, shape.head_dim, 16, n_blocks,
                   max_sessions=n_sessions, max_batch_tokens=4096, kv_fill=0xFF)
    pool.sk_pool_set_alloc_order(synth.permutation(gen, n_blocks))
    ref = oracle.OraclePool(shape.dtype, shape.n_q_heads, shape.n_kv_heads, shape.head_dim)
    sids = [pool.sk_session_create() for _ in range(n_sessions)]
    for _ in sids:
        ref.create()
    _grow(pool, ref, sids, lengths, shape, gen)
    _check_caches(pool, ref, sids)
    for step in range(3):
        order = [int(x) for x in synth.permutation(gen, n_sessions)]
        n_app = max(1, n_sessions // 3)
        ops, counts = [], []
        for j, s in enumerate(order):
            if j < n_app:
                ops.append(sk.SK_OP_APPEND); counts.append(synth.randint(gen, 128, 300))
            else:
                ops.append(sk.SK_OP_QUERY_B if j % 2 else sk.SK_OP_QUERY_A); counts.append(synth.randint(gen, 8, 64))
        if step == 2:
            counts[-1] = 0                      # an empty item is legal
        cu = np.concatenate([[0], np.cumsum(counts)]).astype(np.int32)
        q, k, v = synth.draw_qkv(gen, int(cu[-1]), shape)
        out, lse = pool.sk_batch_step(order, ops, cu, dev(q), dev(k), dev(v))
        ro, rl = ref.batch_step(order, ops, cu, synth.to_raw(q), synth.to_raw(k), synth.to_raw(v))
        compare("step %d" % step, out, lse, ro, rl, shape.dtype)
        for s in order:
            assert pool.sk_session_length(s) == ref.sessions[s].length
    _check_caches(pool, ref, sids)
    # blocks no session owns still hold the canary bytes; so does nothing else get written
    owned = set()
    for sid in sids:
        owned.update(pool.sk_session_block_table(sid))
    torch.cuda.synchronize()
    mem = pool.kv_mem
    free = [b for b in range(n_blocks) if b not in owned][:50]
    for b in free:
        for h in (0, shape.n_kv_heads - 1):
            a = pool.sk_pool_element_offset(b, h, False, 0, 0)
            e = pool.sk_pool_element_offset(b, h, True, 15, shape.head_dim - 1)
            assert bool((mem[a:e] == 0xFF).all()), "block %d was written" % b


@pytest.mark.parametrize("tokens", [3, 40, 70])
def test_step_over_sessions_at_the_edges_of_a_piece(tokens):
    """Cached lengths around the shortest piece a tile is cut into (256 keys), empty sessions and one much
    longer than the others, so that whole pieces, remainders and single-piece tiles (written directly)
    meet in one launch; 3 / 40 / 70 tokens take the 64-, 256- and 256-row kernels."""
    shape = synth.CFG4
    gen = synth.generator(4, stream=500 + tokens)
    lengths = [0, 1, 64, 255, 256, 257, 512, 513, 6000, 0]
    n = len(lengths)
    pool = sk.Pool(shape.dtype, shape.n_q_heads, shape.n_kv_heads, shape.head_dim, 16, sum(lengths) // 16 + 120, max_sessions=n,
                   max_batch_tokens=2048, kv_fill=0xFF)
    ref = oracle.OraclePool(shape.dtype, shape.n_q_heads, shape.n_kv_heads, shape.head_dim)
    sids = [pool.sk_session_create() for _ in range(n)]
    for _ in sids:
        ref.create()
    _grow(pool, ref, sids, lengths, shape, gen)
    ops = [sk.SK_OP_QUERY_B] * (n - 2) + [sk.SK_OP_QUERY_A, sk.SK_OP_APPEND]
    for step in range(2):
        cu = np.arange(n + 1, dtype=np.int32) * tokens
        q, k, v = synth.draw_qkv(gen, int(cu[-1]), shape)
        out, lse = pool.sk_batch_step(sids, ops, cu, dev(q), dev(k), dev(v))
        ro, rl = ref.batch_step(sids, ops, cu, synth.to_raw(q), synth.to_raw(k), synth.to_raw(v))
        compare("step %d" % step, out, lse, ro, rl, shape.dtype)
        ops = [sk.SK_OP_APPEND, sk.SK_OP_QUERY_A] * (n // 2)
    _check_caches(pool, ref, sids)


def test_batch_errors_leave_state_unchanged():
    shape = synth.CFG4
    gen = synth.generator(4, stream=77)
    pool = sk.Pool(shape.dtype, shape.n_q_heads, shape.n_kv_heads, shape.head_dim, 16, 12, max_sessions=3,
                   max_batch_tokens=512)
    a, b, c = (pool.sk_session_create() for _ in range(3))
    q, k, v = (dev(t) for t in synth.draw_qkv(gen, 200, shape))
    pool.sk_session_append(a, q[:64], k[:64], v[:64])            # 4 blocks
    state = lambda: ([pool.sk_session_length(s) for s in (a, b, c)], pool.sk_pool_blocks_free())
    before = state()
    with pytest.raises(sk.SkError) as e:                          # needs 5 + 5 blocks, 8 free
        pool.sk_batch_step([a, b], [sk.SK_OP_APPEND, sk.SK_OP_APPEND], [0, 80, 160], q, k, v)
    assert e.value.status == sk.SK_E_NOMEM and state() == before
    with pytest.raises(sk.SkError) as e:                          # same session twice
        pool.sk_batch_step([a, a], [sk.SK_OP_QUERY_A, sk.SK_OP_QUERY_A], [0, 8, 16], q, k, v)
    assert e.value.status == sk.SK_E_INVAL and state() == before
    with pytest.raises(sk.SkError) as e:                          # cache-only query on an empty session
        pool.sk_batch_step([a, b], [sk.SK_OP_APPEND, sk.SK_OP_QUERY_A], [0, 16, 24], q, k, v)
    assert e.value.status == sk.SK_E_EMPTY and state() == before
    with pytest.raises(sk.SkError) as e:
        pool.sk_batch_step([a, 7], [sk.SK_OP_QUERY_A, sk.SK_OP_QUERY_A], [0, 8, 16], q, k, v)
    assert e.value.status == sk.SK_E_BADSESSION and state() == before
    pool.sk_batch_step([b, a], [sk.SK_OP_APPEND, sk.SK_OP_QUERY_B], [0, 100, 130], q, k, v)
    assert state() == ([64, 100, 0], 1)


@pytest.mark.parametrize("n,P,NQ,Sfx", [(700, 16, 6, 8), (1300, 5, 3, 3), (130, 0, 4, 8), (0, 16, 2, 8), (900, 40, 2, 20)])
def test_shared_prefix_question_batch(n, P, NQ, Sfx):
    """Registered-question batch at the 70B-layer shape (64/8 heads): prefix rows once, suffix rows
    per question; equal to the oracle's independent evaluations, and nothing is committed."""
    shape = synth.CFG5
    gen = synth.generator(5, stream=n + P)
    pool = sk.Pool(shape.dtype, shape.n_q_heads, shape.n_kv_heads, shape.head_dim, 16, n // 16 + 8, max_sessions=1,
                   kv_fill=0xFF)
    ref = oracle.OracleSession(shape.dtype, shape.n_q_heads, shape.n_kv_heads, shape.head_dim)
    sid = pool.sk_session_create()
    if n:
        q, k, v = synth.draw_qkv(gen, n, shape)
        pool.sk_session_append(sid, None, dev(k), dev(v))
        ref.K, ref.V = synth.to_raw(k), synth.to_raw(v)
    qp, kp, vp = synth.draw_qkv(gen, P, shape)
    qs, ks, vs = synth.draw_qkv(gen, NQ * Sfx, shape)
    r4 = lambda t, H: t.reshape(NQ, Sfx, H, shape.head_dim)
    before = pool.kv_mem.clone()
    op, lp, os_, ls = pool.sk_session_query_shared_prefix(
        sid, dev(qp) if P else None, dev(kp) if P else None, dev(vp) if P else None,
        dev(r4(qs, shape.n_q_heads)), dev(r4(ks, shape.n_kv_heads)), dev(r4(vs, shape.n_kv_heads)))
    rop, rlp, ros, rls = ref.query_shared_prefix(
        synth.to_raw(qp), synth.to_raw(kp), synth.to_raw(vp),
        synth.to_raw(qs).reshape(NQ, Sfx, shape.n_q_heads, -1), synth.to_raw(ks).reshape(NQ, Sfx, shape.n_kv_heads, -1),
        synth.to_raw(vs).reshape(NQ, Sfx, shape.n_kv_heads, -1))
    if P:
        compare("prefix rows", op, lp, rop, rlp, shape.dtype)
    compare("suffix rows", os_, ls, ros.reshape(NQ * Sfx, shape.n_q_heads, -1), rls.reshape(NQ * Sfx, -1), shape.dtype)
    torch.cuda.synchronize()
    assert torch.equal(before, pool.kv_mem) and pool.sk_session_length(sid) == n


@pytest.mark.parametrize("n,P,NQ,Sfx,packed", [(700, 16, 6, 8, True), (0, 16, 9, 16, False), (330, 40, 3, 32, False), (65, 0, 5, 5, False),
                                               (33, 16, 24, 16, True), (2000, 20, 9, 8, True)])
def test_shared_prefix_question_batch_head_dim_64(n, P, NQ, Sfx, packed):
    """Questions of a head_dim 64 layer, packed into 256-row tiles where their rows allow it and that is expected to end earlier."""
    shape = synth.Shape("bf16", 32, 8, 64)
    gen = synth.generator(5, stream=3000 + n + P)
    pool = sk.Pool(shape.dtype, shape.n_q_heads, shape.n_kv_heads, shape.head_dim, 16, n // 16 + 8, max_sessions=1, kv_fill=0xFF)
    ref = oracle.OracleSession(shape.dtype, shape.n_q_heads, shape.n_kv_heads, shape.head_dim)
    sid = pool.sk_session_create()
    if n:
        q, k, v = synth.draw_qkv(gen, n, shape)
        pool.sk_session_append(sid, None, dev(k), dev(v))
        ref.K, ref.V = synth.to_raw(k), synth.to_raw(v)
    qp, kp, vp = synth.draw_qkv(gen, P, shape)
    qs, ks, vs = synth.draw_qkv(gen, NQ * Sfx, shape)
    r4 = lambda t, H: t.reshape(NQ, Sfx, H, shape.head_dim)
    op, lp, os_, ls = pool.sk_session_query_shared_prefix(
        sid, dev(qp) if P else None, dev(kp) if P else None, dev(vp) if P else None,
        dev(r4(qs, shape.n_q_heads)), dev(r4(ks, shape.n_kv_heads)), dev(r4(vs, shape.n_kv_heads)))
    tiles = -(-NQ * Sfx * 4 // 256) if packed else NQ * -(-Sfx * 4 // 128)
    assert pool.sk_pool_last_launch()["row_tiles"] == tiles + -(-P * 4 // 128)
    rop, rlp, ros, rls = ref.query_shared_prefix(
        synth.to_raw(qp), synth.to_raw(kp), synth.to_raw(vp),
        synth.to_raw(qs).reshape(NQ, Sfx, shape.n_q_heads, -1), synth.to_raw(ks).reshape(NQ, Sfx, shape.n_kv_heads, -1),
        synth.to_raw(vs).reshape(NQ, Sfx, shape.n_kv_heads, -1))
    if P:
        compare("prefix rows", op, lp, rop, rlp, shape.dtype)
    compare("suffix rows", os_, ls, ros.reshape(NQ * Sfx, shape.n_q_heads, -1), rls.reshape(NQ * Sfx, -1), shape.dtype)


@pytest.mark.parametrize("n,P,NQ,Sfx", [(2000, 20, 9, 8), (2000, 16, 5, 16), (33, 16, 24, 16)])
def test_infinite_value_of_one_question_stays_with_it_head_dim_64(n, P, NQ, Sfx):
    """Questions packed into 256-row tiles: an infinite value of one question's suffix is met by no row of another question,
    not even with a weight of 0."""
    shape = synth.Shape("bf16", 32, 8, 64)
    gen = synth.generator(5, stream=3100 + n + P)
    pool = sk.Pool(shape.dtype, shape.n_q_heads, shape.n_kv_heads, shape.head_dim, 16, n // 16 + 8, max_sessions=1)
    sid = pool.sk_session_create()
    if n:
        _, k, v = synth.draw_qkv(gen, n, shape)
        pool.sk_session_append(sid, None, dev(k), dev(v))
    qp, kp, vp = (dev(x) if P else None for x in synth.draw_qkv(gen, P, shape))
    r4 = lambda t: dev(t.reshape(NQ, Sfx, t.shape[1], shape.head_dim))
    qs, ks, vs = (r4(x) for x in synth.draw_qkv(gen, NQ * Sfx, shape))
    hit = NQ // 2
    vs[hit, 0, :, 7] = 0.0
    planted = vs.clone()
    planted[hit, 0, :, 7] = float("inf")
    a = pool.sk_session_query_shared_prefix(sid, qp, kp, vp, qs, ks, vs)
    b = pool.sk_session_query_shared_prefix(sid, qp, kp, vp, qs, ks, planted)
    assert pool.sk_pool_last_launch()["row_tiles"] == (1 if P else 0) + -(-NQ * Sfx * 4 // 256)       # packed
    others = [j for j in range(NQ) if j != hit]
    assert torch.equal(a[2][others], b[2][others]) and torch.equal(a[3], b[3])
    assert not torch.isfinite(b[2][hit, :, :, 7]).any()
    if P:
        assert torch.equal(a[0], b[0]) and torch.equal(a[1], b[1])


def test_piece_lengths_behind_a_repeated_one_are_looked_at():
    """The lengths a launch's tiles may be cut into are multiples of 64, at least 256: 3,143 keys in 10 pieces and in 12 are pieces of
    320 keys both times, and the length chosen here, 256, comes behind them."""
    shape = synth.Shape("bf16", 64, 8, 128)
    n, P, NQ, Sfx = 3143, 16, 26, 16
    gen = synth.generator(5, stream=3900)
    pool = sk.Pool(shape.dtype, shape.n_q_heads, shape.n_kv_heads, shape.head_dim, 16, n // 16 + 8, max_sessions=1)
    ref = oracle.OracleSession(shape.dtype, shape.n_q_heads, shape.n_kv_heads, shape.head_dim)
    sid = pool.sk_session_create()
    _, k, v = synth.draw_qkv(gen, n, shape)
    pool.sk_session_append(sid, None, dev(k), dev(v))
    ref.K, ref.V = synth.to_raw(k), synth.to_raw(v)
    prefix = synth.draw_qkv(gen, P, shape)
    suffix = [x.reshape(NQ, Sfx, x.shape[1], -1) for x in synth.draw_qkv(gen, NQ * Sfx, shape)]
    op, lp, os_, ls = pool.sk_session_query_shared_prefix(sid, *(dev(x) for x in prefix), *(dev(x) for x in suffix))
    geo = pool.sk_pool_last_launch()
    assert geo["n_splits"] == -(-n // 256) and geo["workgroups"] == 8 * 3 * 13, geo
    rop, rlp, ros, rls = ref.query_shared_prefix(*(synth.to_raw(x) for x in prefix), *(synth.to_raw(x) for x in suffix))
    compare("prefix rows", op, lp, rop, rlp, shape.dtype)
    compare("suffix rows", os_, ls, ros.reshape(NQ * Sfx, 64, -1), rls.reshape(NQ * Sfx, -1),
            shape.dtype)


@pytest.mark.parametrize("n,T,N,variant", [(304, 363, 3, 3), (888, 137, 12, 1), (90, 37, 12, 3)])
def test_head_dim_64_steps_in_both_tile_heights(n, T, N, variant):
    """A step's items of more than 128 rows go into tiles of 256 rows, or of 128 where the launches are expected to end earlier:
    appends and both kinds of queries, beside an item of few rows."""
    shape = synth.Shape("bf16", 32, 8, 64)
    gen = synth.generator(4, stream=400 + T)
    pool = sk.Pool(shape.dtype, shape.n_q_heads, shape.n_kv_heads, shape.head_dim, 16, (N + 1) * ((n + T) // 16 + 2), max_sessions=N + 1,
                   max_batch_tokens=2048, kv_fill=0xFF)
    ref = oracle.OraclePool(shape.dtype, shape.n_q_heads, shape.n_kv_heads, shape.head_dim)
    sids = [pool.sk_session_create() for _ in range(N + 1)]
    for _ in sids:
        ref.create()
    _grow(pool, ref, sids, [n] * (N + 1), shape, gen)
    ops = [(sk.SK_OP_APPEND, sk.SK_OP_QUERY_B, sk.SK_OP_QUERY_A)[i % 3] for i in range(N + 1)]
    for counts in ([T] * N + [0], [T] * N + [5]):
        cu = np.concatenate([[0], np.cumsum(counts)]).astype(np.int32)
        q, k, v = synth.draw_qkv(gen, int(cu[-1]), shape)
        out, lse = pool.sk_batch_step(sids, ops, cu, dev(q), dev(k), dev(v))
        assert pool.sk_pool_last_launch()["kernel_variant"] == variant or counts[-1]
        ro, rl = ref.batch_step(sids, ops, cu, synth.to_raw(q), synth.to_raw(k), synth.to_raw(v))
        compare("step of %s" % counts, out, lse, ro, rl, shape.dtype)
    _check_caches(pool, ref, sids)


@pytest.mark.parametrize("hq,hkv,d", [(32, 8, 128), (14, 2, 64)])
def test_cache_policy_of_lone_tiles_in_batched_steps(hq, hkv, d):
    """Items of one row tile load their keys non-temporal where a step reads enough of them (here: always, and never); several tiles of a
    session never do.  The same bits either way, at both sides of the 64- and 128-row tiles and with evicted keys."""
    shape = synth.Shape("bf16", hq, hkv, d)
    gen = synth.generator(4, stream=4000 + d)
    G = hq // hkv
    counts = [1, 64 // G, 64 // G + 1, 128 // G, 128 // G + 1, 2 * (128 // G) + 3]
    lengths = [1, 63, 700, 1025, 333, 64]
    pools = [Pair(shape, block_tokens=16, n_blocks=400, max_sessions=len(counts), max_batch_tokens=2048, env=env).pool
             for env in ({"SK_STREAM_MIN_TOKENS": "0"}, {"SK_NO_STREAM_LOADS": "1"}, None)]
    sids = [[p.sk_session_create() for _ in counts] for p in pools]
    for i, n in enumerate(lengths):
        _, k, v = [dev(t) for t in synth.draw_qkv(gen, n, shape)]
        for p, s in zip(pools, sids):
            p.sk_session_append(s[i], None, k, v)
            if n == 700:
                p.sk_session_freeze(s[i], 5)
                p.sk_session_evict_oldest(s[i], 100)
    cu = np.concatenate([[0], np.cumsum(counts)]).astype(np.int32)
    for ops in ([sk.SK_OP_QUERY_B] * len(counts), [sk.SK_OP_QUERY_A] * len(counts), [sk.SK_OP_APPEND, sk.SK_OP_QUERY_B] * (len(counts) // 2)):
        q, k, v = [dev(t) for t in synth.draw_qkv(gen, int(cu[-1]), shape)]
        results = [p.sk_batch_step(s, ops, cu, q, k, v) for p, s in zip(pools, sids)]
        for out, lse in results[1:]:
            assert torch.equal(out, results[0][0]) and torch.equal(lse, results[0][1]), ops


@pytest.mark.parametrize("hq,hkv,d,dtype", [(32, 8, 128, "bf16"), (16, 2, 64, "bf16"), (4, 4, 64, "f32")])
def test_lists_that_the_scatter_launch_carries(hq, hkv, d, dtype):
    """Lists beyond 16 KiB are copied to the workspace by items of the scatter launch, 4 KiB a workgroup: steps with something to scatter and
    without, few KV heads (several such items) and more, then questions without a prefix (whose own scatter list is empty)."""
    shape = synth.Shape(dtype, hq, hkv, d)
    gen = synth.generator(4, stream=5000 + hq + d)
    n_sessions, T = {8: (14, 40), 4: (24, 40), 2: (48, 80)}[hkv]
    pr = Pair(shape, block_tokens=16, n_blocks=n_sessions * 60, max_sessions=n_sessions, max_batch_tokens=4096)
    sids = [pr.create() for _ in range(n_sessions)]
    for i, s in enumerate(sids):
        _, k, v = synth.draw_qkv(gen, 500 + 7 * i, shape)
        pr.pool.sk_session_append(s, None, dev(k), dev(v))
        pr.oracles[s].K, pr.oracles[s].V = synth.to_raw(k), synth.to_raw(v)
    cu = np.arange(n_sessions + 1, dtype=np.int32) * T
    for op in (sk.SK_OP_QUERY_A, sk.SK_OP_QUERY_B):
        q, k, v = synth.draw_qkv(gen, n_sessions * T, shape)
        own = (dev(k), dev(v)) if op == sk.SK_OP_QUERY_B else (None, None)
        out, lse = pr.pool.sk_batch_step(sids, [op] * n_sessions, cu, dev(q), *own)
        assert pr.pool.sk_pool_last_launch()["workgroups"] * 88 > 16384
        for i in (0, n_sessions // 2, n_sessions - 1):
            a, b = cu[i], cu[i + 1]
            ro, rl = pr.oracles[sids[i]].query(synth.to_raw(q[a:b]), *((synth.to_raw(k[a:b]), synth.to_raw(v[a:b])) if own[0] is not None else ()))
            compare("op %d session %d" % (op, i), out[a:b], lse[a:b], ro, rl, dtype)
    NQ, Sfx = (40 if hkv > 2 else 120), 8
    qs, ks, vs = synth.draw_qkv(gen, NQ * Sfx, shape)
    r4 = lambda t: t.reshape(NQ, Sfx, t.shape[1], d)
    _, _, os_, ls = pr.pool.sk_session_query_shared_prefix(sids[-1], None, None, None, dev(r4(qs)), dev(r4(ks)), dev(r4(vs)))
    for j in (0, NQ - 1):
        a, b = j * Sfx, (j + 1) * Sfx
        ro, rl = pr.oracles[sids[-1]].query(*[synth.to_raw(t[a:b]) for t in (qs, ks, vs)])
        compare("question %d" % j, os_[j], ls[j], ro, rl, dtype)
