"""Probe sequences of the block index and of recently_evicted on the GPU
against the oracle: every block's hash has the same home slot, a few slots
before the end of both tables, so each search runs over many groups of slots,
past deleted and stale ones and around the table's end."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

import synth  # noqa: E402
from harness import Pair, say  # noqa: E402
from paper_2605_18825_amd import api  # noqa: E402


def hashes_at_home(back, n, spread):
    """n distinct hashes whose home slot, in a table of any size up to 2^32, is
    `back` slots before the end (and, with spread, that of the i-th i % spread
    slots later): the home is the upper half of (h ^ h >> 31) * odd."""
    M = 1 << 64
    inv = pow(0x9E3779B97F4A7C15, -1, M)
    out = []
    for i in range(n):
        home = (0xFFFFFFFF - back + (i % spread if spread else 0)) & 0xFFFFFFFF
        z = (((home << 32) | (i + 1)) * inv) % M
        h = z  # undo z = h ^ (h >> 31)
        for _ in range(3):
            h = z ^ (h >> 31)
        out.append(h)
    return np.array(out, np.uint64)


# the last one: dozens of workgroups on every die claim slots of the same few lines at once, so most claims are lost
# and go on from what the compare-and-swap returned
@pytest.mark.parametrize("N,k,back,spread", [(32, 8, 3, 0), (64, 16, 0, 0), (100, 33, 7, 3), (300, 64, 9, 12),
                                             (3000, 1500, 1000, 5)])
def test_one_home_slot(N, k, back, spread):
    cfg = synth.pool_config("large")
    pool = synth.make_pool(cfg, n_blocks=N, seed=N)
    pool["valid"][:] = False
    pool["parent"][:] = -1
    pool["ref_count"][:] = 0
    p = Pair(cfg["kinds"], pool, k, mu=cfg["mu"], sigma=cfg["sigma"], learn=3 | api.LEARN_DECAY_POWER)
    try:
        rng = np.random.default_rng(7 * N)
        H = hashes_at_home(back, 3 * N, spread)
        free, held = np.arange(N), {}
        now = 1000
        for step in range(12):
            say("one home slot: N %d k %d step %d, %d blocks to insert" % (N, k, step, len(free)))
            # hashes not held now: new ones and evicted ones, in any order
            cand = np.array([h for h in H if int(h) not in held.values()], np.uint64)
            hs = rng.permutation(cand)[:len(free)]
            n = len(free)
            ids = rng.permutation(free).astype(np.int32)
            src = rng.integers(0, N, n)
            p.insert(ids, hs, np.full(n, -1, np.int32), np.full(n, now - 1 - step, np.int32), pool["queue"][src],
                     pool["counts"][src], pool["ntok"][src], pool["ob"][src], pool["omax"][src])
            held.update((int(i), int(h)) for i, h in zip(ids, hs))
            p.prefix_match(H.reshape(-1, 1), np.ones(len(H), np.int32), now, api.PM_STATS)
            p.check_counters()
            p.check_pool()
            _, _, dec = p.select(now, k, commit=True)
            free = np.asarray(dec)
            for i in free:
                del held[int(i)]
            p.prefix_match(H.reshape(-1, 1), np.ones(len(H), np.int32), now, api.PM_STATS)
            p.feedback()
            p.check_counters()
            now += 100
        assert sum(p.oc.missed) + p.oc.ev_count > 0
        assert not p.status()
    finally:
        p.close()


@pytest.mark.parametrize("n", [524287, 524288])
def test_bulk_add_and_build(n):
    """Both group sizes of the probes (from 524,288 blocks on another one): a
    cache filled by one Add(), then indexed anew, against the oracle."""
    N = 600011
    cfg = synth.pool_config("large")
    pool = synth.make_pool(cfg, n_blocks=N, seed=n)
    pool["valid"][:] = False
    pool["parent"][:] = -1
    pool["ref_count"][:] = 0
    say("bulk: %d blocks" % n)
    p = Pair(cfg["kinds"], pool, 64, mu=cfg["mu"], sigma=cfg["sigma"])
    try:
        ids = np.random.default_rng(n).permutation(N)[:n].astype(np.int32)
        p.insert(ids, pool["hash"][ids], np.full(n, -1, np.int32), pool["last_access"][ids], pool["queue"][ids],
                 pool["counts"][ids], pool["ntok"][ids], pool["ob"][ids], pool["omax"][ids])
        R, L = synth.make_requests(pool["chains"], 64, 32, 0.9, 9)
        say("bulk: added, matching and selecting")
        p.prefix_match(R, L, pool["now"], api.PM_STATS)
        p.select(pool["now"], 64)
        p.check_counters()
        assert not p.status()
        say("bulk: indexing anew")
        api.sae_index_build(p.ctx)
        p.prefix_match(R, L, pool["now"] + 1, 0)
        assert not p.status()
    finally:
        p.close()
