"""Pool shapes at which the scan's aligned reads, the batched engine's two
selections and the candidate stripes can go wrong, against the oracle:
instances that start at every offset mod 4 and end inside a group of four
blocks, and a k at the limit of the candidate stripes."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

import oracle  # noqa: E402
import synth  # noqa: E402
import torch  # noqa: E402
from harness import Pair, say  # noqa: E402
from paper_2605_18825_amd import api  # noqa: E402
from paper_2605_18825_amd.pool import DevicePool, SelectBuffers  # noqa: E402


def several(n_inst, N, k, flags, layout="large", seed=31, edit=None, k_per=None, mix=None, **prm):
    """n_inst pools in one context: lists, scores, decisions equal the oracle's."""
    cfg = synth.pool_config(layout, n_blocks=N, k=k, **({} if mix is None else dict(mix=mix)))
    Q = len(cfg["kinds"])
    ctx = api.sae_create(n_inst, N, cfg["kinds"], max_k=k)
    try:
        dp, ocs = DevicePool(n_inst, N), []
        for i in range(n_inst):
            pool = synth.make_pool(cfg, seed=seed + i, n_blocks=N)
            if edit is not None:
                edit(pool, np.random.default_rng(seed + i))
            dp.fill_instance(i, pool)
            oc = oracle.OracleCache(N, cfg["kinds"], oracle.Params(Q, mu=cfg["mu"], sigma=cfg["sigma"], K=k, **prm))
            oc.bind(pool["last_access"], pool["queue"], oracle.block_type(pool["counts"]), pool["ntok"], pool["ob"],
                    pool["omax"], pool["valid"], pool["ref_count"], pool["parent"], pool["hash"])
            ocs.append(oc)
        dp.bind(ctx)
        api.sae_index_build(ctx)
        api.sae_set_params(ctx, -1, api.make_params(Q, mu=cfg["mu"], sigma=cfg["sigma"], K=k, **prm))
        out = SelectBuffers(n_inst, Q, k)
        now = synth.pools.NOW
        kd = None if k_per is None else torch.as_tensor(np.asarray(k_per, np.int32)).cuda()
        out.run(ctx, now, k, flags, k_per_inst=kd)
        torch.cuda.synchronize()
        for i, oc in enumerate(ocs):
            ki = k if k_per is None else k_per[i]
            lists, key, dec = oc.score_select(now, ki)
            for q in range(Q):
                c = int(out.count[i, q])
                assert c == len(lists[q]), (i, q, c, len(lists[q]))
                assert np.array_equal(out.victims[i, q, :c].cpu().numpy(), lists[q]), (i, q)
                got = out.scores[i, q, :c].cpu().numpy().view(np.uint32)
                assert np.array_equal(got, key[lists[q]]), (i, q)
            d = int(out.decision_count[i])
            assert np.array_equal(out.decision[i, :d].cpu().numpy(), dec), i
        return api.status_names(api.sae_poll_status(ctx))
    finally:
        api.sae_destroy(ctx)


@pytest.mark.parametrize("N", [1, 2, 3, 5, 255, 257, 1001, 4098, 16387])
def test_scan_instances_at_every_alignment(N):
    say("scan: 5 instances of %d blocks" % N)
    several(5, N, max(1, min(64, N)), api.SS_ENGINE_SCAN)


def test_scan_large_odd_pool():
    """An odd size at which a wave reads several batches."""
    say("scan: 700,001 blocks")
    assert several(1, 700001, 1000, api.SS_ENGINE_SCAN) == []


@pytest.mark.parametrize("N", [16384, 40003])
def test_batched_small_k_under_a_large_max_k(N):
    """max_k leaves no room for its lists and the streaming list together:
    instances with a small k stream, the ones with a large k use the cache."""
    say("batched: %d blocks, max_k 2,048" % N)
    several(3, N, 2048, api.SS_ENGINE_BATCHED, k_per=[300, 2048, 1])


@pytest.mark.parametrize("N,k,mix", [(300001, 1000, None), (262144, 4096, [0.6, 0.1, 0.1, 0.1, 0.1]),
                                     (1048576, 300, [0.96, 0.01, 0.01, 0.01, 0.01])])
def test_equal_keys_in_id_order(N, k, mix):
    """Every queue's keys are equal per type, so its candidates are the lowest
    ids, all in a few workgroups of the scan: they take several pieces of their
    stripes, the overflow list where a buffer is full, and splits by value in
    the ranking."""
    def edit(pool, rng):
        pool["last_access"][:] = synth.pools.NOW - 5000

    say("equal keys: %d blocks, k %d" % (N, k))
    assert several(1, N, k, api.SS_ENGINE_SCAN, edit=edit, mix=mix) == []


@pytest.mark.parametrize("N,k,mix", [(300001, 1000, None), (1048576, 300, [0.96, 0.01, 0.01, 0.01, 0.01])])
def test_equal_keys_with_outliers(N, k, mix):
    """As above, with a few blocks decades older or newer and a few partly
    filled ones, so that splits by value also meet ranges that are empty but
    for their ends."""
    def edit(pool, rng):
        pool["last_access"][:] = synth.pools.NOW - 5000
        pool["last_access"][rng.choice(N, 40, replace=False)] = synth.pools.NOW - 900000
        pool["last_access"][rng.choice(N, 40, replace=False)] = synth.pools.NOW - 1
        pool["ntok"][rng.choice(N, 40, replace=False)] = 15
        pool["ntok"][rng.choice(N, 10, replace=False)] = 1

    say("equal keys and outliers: %d blocks, k %d" % (N, k))
    assert several(1, N, k, api.SS_ENGINE_SCAN, edit=edit, mix=mix) == []


def test_largest_k_without_fallback():
    """k = 8,192 on 4M blocks: about 16,000 candidates per queue, more than the
    stripes alone hold; their overflow list takes the rest and the exact slow
    path stays out."""
    cfg = synth.pool_config("large")
    say("k = 8,192: generating pool")
    pool = synth.make_pool(cfg, seed=88)
    p = Pair(cfg["kinds"], pool, 8192, mu=cfg["mu"], sigma=cfg["sigma"], K=8192)
    try:
        for t in (0, 400, 800):
            say("k = 8,192: score_select")
            p.select(pool["now"] + t, 8192)
        assert not p.status()
    finally:
        p.close()


def newest_last(pool, rng):
    """Every block older than the ones before it: each one is among the k smallest so far."""
    pool["last_access"] = np.sort(pool["last_access"])[::-1].copy()


def newest_first(pool, rng):
    pool["last_access"] = np.sort(pool["last_access"])


def clusters(pool, rng):
    pool["last_access"] = (synth.pools.NOW - 1000 * rng.integers(1, 13, pool["n_blocks"])).astype(np.int32)


def late_queue(pool, rng):
    """Queue 2 only in the last tenth of the pool, the evict-first queue only in the first blocks."""
    n, q = pool["n_blocks"], pool["queue"]
    q[: n - n // 10][q[: n - n // 10] == 2] = 3
    q[64:][q[64:] == 0] = 4


def edges(pool, rng):
    """Blocks accessed now and in the future, partly filled blocks, offsets at their ends."""
    n = pool["n_blocks"]
    pool["last_access"][rng.random(n) < 0.3] = synth.pools.NOW
    pool["last_access"][rng.random(n) < 0.05] = synth.pools.NOW + 5
    pool["ntok"] = rng.integers(1, 17, n).astype(np.int32)
    pool["ob"] = np.where(rng.random(n) < 0.5, pool["omax"], 0).astype(np.int32)


# the batched engine around and above 16,384 blocks, streamed (small k) and cached, every alignment
@pytest.mark.parametrize("N,k", [(16384, 1), (16385, 64), (16387, 819), (16383, 64), (40001, 819), (65535, 257),
                                 (65536, 256), (65536, 820)])
def test_batched_streaming_sizes(N, k):
    say("batched: 3 instances of %d blocks, k %d" % (N, k))
    assert several(3, N, k, api.SS_ENGINE_BATCHED) == []


@pytest.mark.parametrize("edit", [newest_last, newest_first, clusters, late_queue, edges])
def test_batched_streaming_orders(edit):
    say("batched: %s" % edit.__name__)
    st = several(3, 30003, 300, api.SS_ENGINE_BATCHED, edit=edit, k_per=[300, 0, 7])
    assert set(st) <= {"FUTURE_ACCESS"}
    say("scan: %s" % edit.__name__)
    several(3, 30003, 300, api.SS_ENGINE_SCAN, edit=edit, k_per=[300, 0, 7])


# on both sides of the rule for streaming (5 queues) and of the largest pool cached in LDS
@pytest.mark.parametrize("N,k", [(12001, 50), (16383, 128), (16384, 128), (16384, 129), (16385, 20), (24003, 57),
                                 (24003, 58), (30002, 228), (30002, 229), (40001, 357), (40001, 358), (65536, 585),
                                 (65536, 586)])
def test_batched_streaming_rule(N, k):
    say("batched: 2 instances of %d blocks, k %d" % (N, k))
    assert several(2, N, k, api.SS_ENGINE_BATCHED) == []


@pytest.mark.parametrize("edit", [newest_last, newest_first, clusters, late_queue, edges])
@pytest.mark.parametrize("N,k", [(40003, 350), (65533, 500)])
def test_batched_streaming_orders_large(edit, N, k):
    say("batched: %s, %d blocks, k %d" % (edit.__name__, N, k))
    st = several(3, N, k, api.SS_ENGINE_BATCHED, edit=edit, k_per=[k, 0, 7])
    assert set(st) <= {"FUTURE_ACCESS"}


# A negative queue or type weight makes negative scores, whose keys (the order of the score's bits) have the top bit
# set; -0.0 is one of them.  In one queue, in all, and in part of each.
@pytest.mark.parametrize("alpha,w", [([1, 1, -2, 1, 1], 1), ([-1, -1, -1, -3, -2], 1), (1, [-1, -1, 2, -1, -1]),
                                     ([1, -0.0, 1, 1, -0.0], 1)])
@pytest.mark.parametrize("k", [40, 300])
def test_negative_weights(alpha, w, k):
    for name, fl in (("batched", api.SS_ENGINE_BATCHED), ("scan", api.SS_ENGINE_SCAN)):
        say("%s: alpha %s w %s k %d" % (name, alpha, w, k))
        assert several(2, 40003, k, fl, alpha=alpha, w=w) == []


# Few buckets per queue (28 to 64 of them with one block in 64 sampled, a single one where the sample holds none):
# the cuts of the candidate ranges on both sides of the ranking's workgroups.
@pytest.mark.parametrize("k", [1, 64, 150, 200, 260])
@pytest.mark.parametrize("mix", [None, [0.0001, 0.4, 0.5996, 0.00002, 0.0999]])
def test_scan_few_buckets(k, mix):
    say("scan: 1,048,576 blocks, k %d, mix %s" % (k, mix))
    assert several(1, 1048576, k, api.SS_ENGINE_SCAN, mix=mix) == []


# equal keys in clusters: ranked by comparison, refined by a wave (from 65) or by the workgroup (from 513)
@pytest.mark.parametrize("size", [64, 65, 130, 512, 513, 1500])
def test_scan_clusters_of_equal_keys(size):
    def same_time(pool, rng):
        n = pool["n_blocks"]
        g = rng.permutation(n) // (4 * size)  # about `size` of them in each of the larger queues
        pool["last_access"] = (synth.pools.NOW - 50 * (1 + g)).astype(np.int32)

    say("scan: clusters of %d" % size)
    several(2, 40009, 3000, api.SS_ENGINE_SCAN, edit=same_time)


@pytest.mark.parametrize("kinds", ["E", "L", "ER", "RS", "ELL", "LSRLSRLS", "ERSLRSLL"])
@pytest.mark.parametrize("k", [1, 700, 4000])
def test_scan_queue_counts(kinds, k):
    """One to eight queues, with and without an evict-first one, of very unequal sizes (one empty, one of a few
    blocks): the merged bucket ends and the candidate ranges of every combination."""
    names = dict(E=api.KIND_EVICT_FIRST, L=api.KIND_LOGNORMAL, R=api.KIND_RECENCY, S=api.KIND_STRUCTURAL)
    Q = len(kinds)
    pool = synth.make_pool(synth.pool_config("large"), n_blocks=50021, seed=100 * Q + k)
    rng = np.random.default_rng(k)
    share = np.array([0.6 ** q for q in range(Q)])
    if Q >= 3:
        share[Q - 1] = 0.0
    pool["queue"] = rng.choice(Q, 50021, p=share / share.sum()).astype(pool["queue"].dtype)
    if Q >= 3:
        pool["queue"][rng.choice(50021, 40, replace=False)] = Q - 2
    p = Pair([names[x] for x in kinds], pool, k, mu=[5.0 + 0.5 * q for q in range(Q)], sigma=[1.0] * Q, K=k)
    try:
        for t in (0, 300):
            say("scan: queues %s, k %d" % (kinds, k))
            p.select(pool["now"] + t, k, flags=api.SS_ENGINE_SCAN)
        assert not p.status()
    finally:
        p.close()


# Every queue's bound admits all of its blocks (its last bucket end is the largest value there is, as in the
# other queues) and k takes every evictable block or nearly so: the decision reaches the last merged ends, several
# of which make one share of the ranking.  Evictable blocks per queue, evict-first one first.
@pytest.mark.parametrize("N,sizes", [(20000, [0, 1300, 900, 390]), (20000, [25, 700, 600, 500]),
                                     (20000, [0, 1500, 140]), (20000, [3, 300, 1, 0, 2000, 131]),
                                     (20000, [0, 40, 30, 0, 20]), (4096, [0, 1100, 800, 600]), (300, [10, 60, 50, 40])])
def test_scan_takes_every_block(N, sizes):
    kinds = [api.KIND_EVICT_FIRST] + [[api.KIND_LOGNORMAL, api.KIND_RECENCY, api.KIND_STRUCTURAL][q % 3]
                                      for q in range(len(sizes) - 1)]
    Q, total = len(sizes), sum(sizes)
    pool = synth.make_pool(synth.pool_config("large"), n_blocks=N, seed=N + total)
    rng = np.random.default_rng(total)
    leaves = np.setdiff1d(np.arange(N), pool["parent"])
    free = rng.permutation(leaves)[:total]
    pool["ref_count"][:] = 1
    pool["ref_count"][free] = 0
    pool["queue"][:] = 1
    pool["queue"][free] = np.repeat(np.arange(Q), sizes)
    fl = api.SS_ENGINE_SCAN if N <= 16384 else 0  # a single larger cache is scanned without being asked
    p = Pair(kinds, pool, 4096, mu=[6.0 + q for q in range(Q)], sigma=[1.2] * Q, K=4096)
    R, L = synth.make_requests(pool["chains"], 8, 16, 0.9, 3)
    try:
        # the scores and with them the merged ends change from call to call
        for t, k in ((0, total), (70000, total + 9), (400000, total - 2), (3000000, total)):
            say("scan: %d blocks, evictable %s, k %d" % (N, sizes, k))
            p.out.decision.fill_(-1)
            p.select(pool["now"] + t, k, flags=fl)
        p.out.decision.fill_(-1)
        p.match_select(R, L, pool["now"] + 4000000, api.PM_TOUCH, pool["now"] + 4000000, total, fl)
        p.out.decision.fill_(-1)
        p.select(pool["now"] + 5000000, total - 4, flags=fl, commit=True)
        p.check_pool()
        p.check_counters()
        assert not p.status()
    finally:
        p.close()


# one wave, one workgroup round, the LDS key cache's limit and the sorts' segment sizes
@pytest.mark.parametrize("N,k", [(1, 1), (63, 2), (1024, 128), (1025, 129), (8192, 256), (8193, 100), (9001, 1)])
def test_batched_small_pools(N, k):
    say("batched: 4 instances of %d blocks, k %d" % (N, k))
    several(4, N, k, api.SS_ENGINE_BATCHED)


# the list sorts: whole lists in a wave, up to four runs a list and one element per thread by ranks, then merged runs
# (or, for one short list more than fits, the bitonic network); and the merge of the lists
@pytest.mark.parametrize("kinds", ["L", "RS", "ELR", "ELLR", "ESLLR", "LSRLSRLS"])
@pytest.mark.parametrize("k", [31, 64, 65, 128, 129, 200, 256, 257, 512, 700, 1500])
def test_batched_list_sizes(kinds, k):
    names = dict(E=api.KIND_EVICT_FIRST, L=api.KIND_LOGNORMAL, R=api.KIND_RECENCY, S=api.KIND_STRUCTURAL)
    Q = len(kinds)
    pool = synth.make_pool(synth.pool_config("large"), n_blocks=6007, seed=50 * Q + k)
    rng = np.random.default_rng(k)
    pool["queue"] = rng.integers(0, Q, 6007).astype(pool["queue"].dtype)
    p = Pair([names[x] for x in kinds], pool, k, mu=[5.0 + 0.5 * q for q in range(Q)], sigma=[1.0] * Q, K=k)
    try:
        for t in (0, 300):
            say("batched: queues %s, k %d" % (kinds, k))
            p.select(pool["now"] + t, k, flags=api.SS_ENGINE_BATCHED)
        assert not p.status()
    finally:
        p.close()


@pytest.mark.parametrize("n_inst,N,k", [(300, 1501, 40), (270, 24601, 60)])
def test_batched_more_caches_than_compute_units(n_inst, N, k):
    """Workgroups that start when others have ended, with the key cache in LDS and streamed."""
    say("batched: %d caches of %d blocks" % (n_inst, N))
    assert several(n_inst, N, k, api.SS_ENGINE_BATCHED) == []
