"""Measured cases of the eviction hot path, through the library's public entry points.

Six kinds of case:
  select   sae_score_select without commit: what would be evicted now
  step     a serving step on a full cache: sae_match_select (touch, stats, commit), sae_feedback_update,
           sae_insert_blocks into the freed slots (and sae_ref_blocks with "hold"), time moving on every pass
  engine   the same step through the host block manager adapter (DeviceBackend): host arrays in, decisions out
  match    sae_prefix_match of a request batch
  predict  the session predictor on a batch of hidden states

Pools follow the distributions of synth/pools.py (drawn on the GPU here, so that a large one is quick to
make): Dirichlet(0.5) token types, last access uniform over 1,000 s, 30 % non-leaf and 10 % referenced
blocks, chained requests of which 60 % start with a cached prefix.
"""
import math

import numpy as np
import torch

from paper_2605_18825_amd import api
from paper_2605_18825_amd.engine import DeviceBackend
from paper_2605_18825_amd.pool import DevicePool, SelectBuffers

NOW = 1_000_000  # ticks (ms)
STEP_TICKS = 1000
EF, STRUCT, LN, REC = 0, 1, 2, 3
MU_CHAT, SIGMA_CHAT = 4.82 + math.log(1000.0), 1.25
MU_AGENT, SIGMA_AGENT = 2.28 + math.log(1000.0), 1.34
# queue layouts: kinds, share of the blocks, mu, sigma
LAYOUTS = {
    "session": ([LN, STRUCT, REC], [0.50, 0.35, 0.15], [MU_CHAT, 0.0, 0.0], [SIGMA_CHAT, 1.0, 1.0]),
    "paper": ([EF, STRUCT, LN, LN], [0.10, 0.40, 0.30, 0.20], [0.0, 0.0, MU_CHAT, MU_AGENT],
              [1.0, 1.0, SIGMA_CHAT, SIGMA_AGENT]),
    "five": ([EF, STRUCT, LN, LN, REC], [0.10, 0.30, 0.30, 0.20, 0.10], [0.0, 0.0, MU_CHAT, MU_AGENT, 0.0],
             [1.0, 1.0, SIGMA_CHAT, SIGMA_AGENT, 1.0]),
}
CHAIN = 8  # blocks of one inserted request tail


def listed():
    return [
        # one small cache asked for its victims: latency of a single call
        dict(name="select_tiny", kind="select", layout="session", inst=1, blocks=4096, k=64, cascade=False),
        # a 36K-token cache behind the host block manager, one request a step
        dict(name="engine_one_cache", kind="engine", inst=1, blocks=2250, k=48, req_len=90),
        # a fleet of such caches stepped together, running requests holding their blocks
        dict(name="step_fleet_small", kind="step", layout="paper", inst=256, blocks=2250, k=64, req=256, req_len=90,
             learn=3, intervals=False, hold=True),
        # one mid-size cache (4M tokens), a batch of 256 requests
        dict(name="step_mid", kind="step", layout="session", inst=1, blocks=262144, k=1024, req=256, req_len=32,
             learn=3, intervals=False, hold=False),
        # the large-pool configuration: 64M tokens, 4,096 requests of 128 hashes
        dict(name="step_large", kind="step", layout="five", inst=1, blocks=4194304, k=4096, req=4096, req_len=128,
             learn=3, intervals=False, hold=False),
        # every learner on, odd sizes
        dict(name="step_learners", kind="step", layout="five", inst=1, blocks=1500007, k=2001, req=1001, req_len=203,
             learn=15, intervals=True, hold=False),
        # the score+select pass alone on the large pool
        dict(name="select_large", kind="select", layout="five", inst=1, blocks=4194304, k=4096, cascade=False),
        # a decision one victim at a time (Algorithm 1 as printed), odd size
        dict(name="select_cascade", kind="select", layout="five", inst=1, blocks=1000003, k=1000, cascade=True),
        # the batched sweep: 256 caches of 1M tokens decided in one call
        dict(name="select_sweep", kind="select", layout="paper", inst=256, blocks=65536, k=256, cascade=False),
        # a scheduler asking what is cached, without touching it
        dict(name="match_large", kind="match", layout="five", inst=1, blocks=4194304, req=4096, req_len=128,
             touch=False, intervals=False, ids=False),
        # session predictor: a full batch of d = 4,096 states, and a small one of a wider model
        dict(name="predict_large", kind="predict", n=4096, d=4096, own_buffer=False),
        dict(name="predict_small", kind="predict", n=37, d=8192, own_buffer=True),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["select", "select", "step", "step", "step", "match", "predict", "engine"])
    if kind == "predict":
        own = rng.random() < 0.5
        return dict(kind=kind, n=_log(rng, 1, 4096), d=256 * rng.randint(4, 16), own_buffer=own)
    if kind == "engine":
        return dict(kind=kind, inst=_log(rng, 1, 16), blocks=_log(rng, 1500, 16000), k=_log(rng, 8, 64),
                    req_len=_log(rng, 16, 200))
    layout = rng.choice(sorted(LAYOUTS))
    if kind == "match":
        touch = rng.random() < 0.5
        iv = touch and rng.random() < 0.5
        return dict(kind=kind, layout=layout, inst=1, blocks=_log(rng, 4096, 4194304), req=_log(rng, 16, 4096),
                    req_len=_log(rng, 8, 128), touch=touch, intervals=iv, ids=iv or rng.random() < 0.5)
    if rng.random() < 0.3:  # a fleet
        inst = _log(rng, 32, 256)
        blocks = _log(rng, 2000, 65536)
        if kind == "step":
            blocks = min(blocks, 16384)
        k = _log(rng, 16, min(256, blocks // 16))
        req = inst
    else:
        inst = 1
        blocks = _log(rng, 4096, 4194304)
        k = _log(rng, 16, min(4096, blocks // 16))
        req = _log(rng, 16, 4096)
    if kind == "select":
        return dict(kind=kind, layout=layout, inst=inst, blocks=blocks, k=k, cascade=rng.random() < 0.25)
    iv = rng.random() < 0.3
    return dict(kind=kind, layout=layout, inst=inst, blocks=blocks, k=k, req=req, req_len=_log(rng, 8, 128),
                learn=15 if iv else 3, intervals=iv, hold=rng.random() < 0.3)


# ------------------------------------------------------------------ inputs
class _Cache:
    """A context and its pool; destroyed with the object."""

    def __init__(self, n_inst, N, kinds, max_k, max_requests):
        self.ctx = api.sae_create(n_inst, N, kinds, max_k=max_k, max_requests=max_requests)
        self.pool = DevicePool(n_inst, N)
        self.pool.bind(self.ctx)

    def __del__(self):
        ctx, self.ctx = getattr(self, "ctx", None), None
        if ctx is not None:
            api.sae_destroy(ctx)


def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed))
    return g


def _hashes(shape, g):
    h = torch.randint(-(1 << 63), (1 << 63) - 1, shape, dtype=torch.int64, device="cuda", generator=g)
    return torch.where((h == 0) | (h == -1), torch.ones_like(h), h)  # the two reserved values


def _blocks(n, mix, g):
    """queue, type, num_tokens, o_b, o_max of n blocks."""
    u = torch.rand(n, device="cuda", generator=g)
    edges = torch.tensor(np.cumsum(mix)[:-1] / np.sum(mix), dtype=torch.float32, device="cuda")
    queue = torch.bucketize(u, edges).to(torch.int32)
    # type of the median token under Dirichlet(0.5) shares (squared normals, unnormalised)
    cum = torch.randn((5, n), device="cuda", generator=g).square()
    for t in range(1, 5):
        cum[t] += cum[t - 1]
    tau = (cum[:4] <= 0.5 * cum[4]).sum(0).to(torch.int32)
    part = torch.randint(1, 17, (n,), device="cuda", generator=g, dtype=torch.int32)
    ntok = torch.where(torch.rand(n, device="cuda", generator=g) < 0.1, part, torch.full_like(part, 16))
    omax = torch.randint(31, 251, (n,), device="cuda", generator=g, dtype=torch.int64)
    ob = torch.minimum((torch.rand(n, device="cuda", generator=g) * (omax + 1)).long(), omax)
    return queue, tau, ntok, ob, omax


def _fill(cache, mix, g):
    p = cache.pool
    I, N = p.n_inst, p.N
    T = I * N
    queue, tau, ntok, ob, omax = _blocks(T, mix, g)
    nonleaf = torch.rand((I, N), device="cuda", generator=g) < 0.3
    # each non-leaf block parents one leaf block of its instance: per instance,
    # the non-leaf blocks in random order, then the leaves in random order
    key = torch.randint(0, 1 << 32, (I, N), dtype=torch.int64, device="cuda", generator=g)
    key += (~nonleaf).long() << 32
    key += torch.arange(I, device="cuda")[:, None] << 33
    order = torch.argsort(key.view(-1)).view(I, N) % N
    del key
    n_nl = nonleaf.sum(1, keepdim=True)
    j = torch.arange(N, device="cuda")[None, :]
    kid = torch.gather(order, 1, (j + n_nl).clamp(max=N - 1))
    has = (j < n_nl) & (j + n_nl < N)
    rows = torch.arange(I, device="cuda")[:, None] * N
    parent = torch.full((T,), -1, dtype=torch.int32, device="cuda")
    parent[(rows + kid)[has]] = order[has].to(torch.int32)
    kids = torch.zeros(T, dtype=torch.int32, device="cuda")
    kids[(rows + order)[has]] = 1
    ref = (torch.rand(T, device="cuda", generator=g) < 0.1).to(torch.int32)
    p.parent.copy_(parent)
    p.child_count.copy_(kids)
    p.ref_count.copy_(ref)
    p.meta.copy_(api.meta_to_u16(api.pack_meta(queue, tau, ntok, valid=True, leaf=(kids == 0), ref=(ref > 0))))
    p.off.copy_(api.off_to_u32(api.pack_off(ob, omax)))
    p.last_access.copy_(torch.randint(0, NOW, (T,), device="cuda", generator=g, dtype=torch.int32))
    p.access_count.copy_(torch.randint(1, 8, (T,), device="cuda", generator=g, dtype=torch.int32))
    p.hash.copy_(_hashes((T,), g))


def _requests(cache, req, L, g):
    """[req, L] hashes, lengths and instances: 60 % start with a cached chain's prefix, the rest are new."""
    p = cache.pool
    inst = torch.arange(req, device="cuda") % p.n_inst
    lens = torch.randint(1, L + 1, (req,), device="cuda", generator=g)
    chains = max(1, p.N // L)
    c = (torch.rand(req, device="cuda", generator=g) * chains).long().clamp(max=chains - 1)
    m = torch.minimum((torch.rand(req, device="cuda", generator=g) * lens).long() + 1, lens)
    m = torch.where(torch.rand(req, device="cuda", generator=g) < 0.6, m, torch.zeros_like(m))
    j = torch.arange(L, device="cuda")[None, :]
    src = (inst * p.N + c * L)[:, None] + j
    cached = p.hash[src.clamp(max=p.n_inst * p.N - 1)]
    h = torch.where(j < m[:, None], cached, _hashes((req, L), g))
    h = torch.where(j < lens[:, None], h, torch.zeros_like(h))
    return h.contiguous(), lens.to(torch.int32), inst.to(torch.int32)


def _cache(case, seed, max_requests=0, learn=3):
    kinds, mix, mu, sigma = LAYOUTS[case["layout"]]
    k = case.get("k", 1)
    g = _gen(seed)
    c = _Cache(case["inst"], case["blocks"], kinds, k, max_requests)
    _fill(c, mix, g)
    api.sae_index_build(c.ctx)
    api.sae_set_params(c.ctx, -1, api.make_params(len(kinds), mu=mu, sigma=sigma, K=k, learn=learn))
    return c, g


def _outputs(n_inst, Q, k):
    out = SelectBuffers(n_inst, Q, k)
    out.per_queue = [out.scores[:, q] for q in range(Q)]  # queues' priorities differ by many orders of magnitude
    return out


def _prepare_step(case, seed):
    c, g = _cache(case, seed, max_requests=case["req"] if case["intervals"] else 0, learn=case["learn"])
    kinds, mix, _, _ = LAYOUTS[case["layout"]]
    I, k = case["inst"], case["k"]
    hashes, lens, inst = _requests(c, case["req"], case["req_len"], g)
    n = I * k
    queue, tau, ntok, ob, omax = _blocks(n, mix, g)
    s = dict(case=case, cache=c, hashes=hashes, lens=lens, inst=inst if I > 1 else None, now=NOW,
             match_len=torch.zeros(case["req"], dtype=torch.int32, device="cuda"),
             ids=torch.empty((case["req"], case["req_len"]), dtype=torch.int32, device="cuda")
             if case["intervals"] else None,
             out=_outputs(I, len(kinds), k),
             flags=api.PM_TOUCH | api.PM_STATS | (api.PM_INTERVALS if case["intervals"] else 0),
             # the step's new blocks: request tails of CHAIN blocks, new contents every pass
             new_hash=_hashes((n,), g), new_la=torch.full((n,), NOW, dtype=torch.int32, device="cuda"),
             new_parent=torch.full((n,), -1, dtype=torch.int32, device="cuda"),
             new_meta=api.meta_to_u16(api.pack_meta(queue, tau, ntok)),
             new_off=api.off_to_u32(api.pack_off(ob, omax)),
             new_inst=torch.arange(I, dtype=torch.int32, device="cuda").repeat_interleave(k) if I > 1 else None,
             held=None, spare=torch.full((n,), -1, dtype=torch.int32, device="cuda"))
    return s


def _prepare_engine(case, seed):
    kinds, mix, mu, sigma = LAYOUTS["paper"]
    I, N, k = case["inst"], case["blocks"], case["k"]
    g = _gen(seed)

    class Backend(DeviceBackend):
        def __del__(self):
            if getattr(self, "ctx", None) is not None:
                self.close()
                self.ctx = None

    be = Backend(I, N, kinds, [0, 1, 2, 3], k, mu, sigma, 32, 3)
    _fill(be, mix, g)
    api.sae_index_build(be.ctx)
    hashes, lens, inst = _requests(be, I, case["req_len"], g)
    h, ln = hashes.cpu().numpy().view(np.uint64), lens.cpu().numpy()
    rng = np.random.default_rng(int(seed))
    n = I * k
    pos = np.tile(np.arange(k, dtype=np.int32), I)
    return dict(case=case, be=be, now=NOW, rng=rng, prompts=[h[i, :ln[i]] for i in range(I)], insts=list(range(I)),
                k=np.full(I, k, np.int32),
                rows=dict(inst=np.repeat(np.arange(I, dtype=np.int32), k), types=rng.integers(0, 5, n),
                          hints=rng.integers(0, 64, n).astype(np.uint8), ob=pos, omax=np.full(n, k + 20, np.int32)))


def _prepare_predict(case, seed):
    n, d = case["n"], case["d"]
    g = _gen(seed)
    x = torch.randn((n, d), device="cuda", generator=g)
    big = torch.randperm(d, device="cuda", generator=g)[:8]
    x[:, big] *= 20.0  # final-layer activations carry a few large channels

    def f(shape, scale):
        return torch.randn(shape, device="cuda", generator=g) * scale
    w = dict(w1=f((256, d), math.sqrt(2.0 / d)).to(torch.bfloat16).view(torch.int16), b1=f((256,), 0.01),
             w2=f((64, 256), math.sqrt(2.0 / 256)), b2=f((64,), 0.01), w3=f((64,), math.sqrt(1.0 / 64)),
             b3=f((1,), 0.01))
    return dict(case=case, h=x.to(torch.bfloat16).view(torch.int16), w=w,
                work=None if case["own_buffer"] else torch.empty((4, n, 256), dtype=torch.float32, device="cuda"),
                logit=torch.empty(n, dtype=torch.float32, device="cuda"),
                pred=torch.empty(n, dtype=torch.uint8, device="cuda"))


def prepare(case, seed):
    kind = case["kind"]
    if kind == "predict":
        return _prepare_predict(case, seed)
    if kind == "engine":
        return _prepare_engine(case, seed)
    if kind == "step":
        return _prepare_step(case, seed)
    if kind == "select":
        c, _ = _cache(case, seed)
        return dict(case=case, cache=c, now=NOW, out=_outputs(case["inst"], len(LAYOUTS[case["layout"]][0]), case["k"]))
    c, g = _cache(case, seed, max_requests=case["req"] if case["intervals"] else 0)
    hashes, lens, _ = _requests(c, case["req"], case["req_len"], g)
    return dict(case=case, cache=c, now=NOW, hashes=hashes, lens=lens,
                match_len=torch.zeros(case["req"], dtype=torch.int32, device="cuda"),
                ids=torch.empty((case["req"], case["req_len"]), dtype=torch.int32, device="cuda") if case["ids"] else None,
                flags=((api.PM_TOUCH | api.PM_STATS) if case["touch"] else 0) |
                (api.PM_INTERVALS if case["intervals"] else 0))


# ------------------------------------------------------------------ one pass
def _selection(out):
    return dict(victims=out.victims, scores=out.per_queue, count=out.count, decision=out.decision,
                decision_count=out.decision_count)


def _run_step(s):
    case, c, out = s["case"], s["cache"], s["out"]
    k, now = case["k"], s["now"]
    if case["hold"] and s["held"] is not None:  # the last step's requests have finished
        api.sae_ref_blocks(c.ctx, s["held"], -1, inst=s["new_inst"])
    out.run_after_match(c.ctx, s["hashes"], s["lens"], now, s["flags"], s["match_len"], now, k, api.SS_COMMIT,
                        matched_ids=s["ids"], inst=s["inst"])
    api.sae_feedback_update(c.ctx, 0)
    ids = out.decision.view(-1)
    full = ids.numel() // CHAIN * CHAIN
    if k % CHAIN == 0 or case["inst"] == 1:  # chains stay inside an instance
        s["new_parent"][:full].view(-1, CHAIN)[:, 1:].copy_(ids[:full].view(-1, CHAIN)[:, :-1])
    api.sae_insert_blocks(c.ctx, ids, s["new_hash"], s["new_parent"], s["new_la"], s["new_meta"], s["new_off"],
                          inst=s["new_inst"])
    if case["hold"]:
        s["spare"].copy_(ids)
        s["held"] = s["spare"]
        api.sae_ref_blocks(c.ctx, s["held"], 1, inst=s["new_inst"])
    # the next step's time and contents
    s["now"] = now + STEP_TICKS
    s["new_la"].add_(STEP_TICKS)
    s["new_hash"].add_(0x1E3779B97F4A7C15)
    p = c.pool
    return dict(_selection(out), match_len=s["match_len"], last_access=p.last_access, meta=p.meta, hash=p.hash,
                child_count=p.child_count, access_count=p.access_count, ref_count=p.ref_count)


def _run_engine(s):
    be, now, f = s["be"], s["now"], s["rows"]
    ml, mids = be.prefix_match(now, s["insts"], s["prompts"])
    dec = be.evict(now, s["k"])
    n = [len(d) for d in dec]
    ids = np.concatenate(dec)
    k = int(s["k"][0])
    keep = np.concatenate([np.arange(i * k, i * k + m) for i, m in enumerate(n)])
    parent = np.concatenate([np.concatenate([[-1], d[:-1]]) for d in dec if len(d)]).astype(np.int32)
    new = {name: v[keep] for name, v in f.items()}
    new.update(ids=ids, parent=parent, hash=s["rng"].integers(1, 1 << 63, len(ids), dtype=np.uint64))
    be.insert(now, new)
    be.feedback()
    s["now"] = now + STEP_TICKS
    matched = np.full((len(mids), s["case"]["req_len"]), -1, np.int32)
    for row, m in zip(matched, mids):
        row[:len(m)] = m
    return dict(match_len=ml, matched=matched, decision=ids, counts=np.array(n, np.int32),
                last_access=be.pool.last_access, meta=be.pool.meta)


def run(s):
    case = s["case"]
    kind = case["kind"]
    if kind == "predict":
        if case["own_buffer"]:
            api.sae_predict_sessions_noalloc(s["h"], s["w"], s["logit"], s["pred"])
        else:
            api.sae_predict_sessions(s["h"], s["w"], s["work"], s["logit"], s["pred"])
        return dict(logit=s["logit"], pred=s["pred"])
    if kind == "step":
        return _run_step(s)
    if kind == "engine":
        return _run_engine(s)
    c = s["cache"]
    s["now"] += 1
    if kind == "select":
        s["out"].run(c.ctx, s["now"], case["k"], api.SS_CASCADE if case["cascade"] else 0)
        return _selection(s["out"])
    api.sae_prefix_match(c.ctx, s["hashes"], s["lens"], s["now"], s["flags"], s["match_len"], matched_ids=s["ids"])
    r = dict(match_len=s["match_len"])
    if s["ids"] is not None:
        r["ids"] = s["ids"]
    if case["touch"]:
        r.update(last_access=c.pool.last_access, access_count=c.pool.access_count)
    return r


# ------------------------------------------------------------------ what a pass cannot do without
def work(case):
    kind = case["kind"]
    if kind == "predict":
        n, d = case["n"], case["d"]
        return dict(bytes=2 * n * d + 2 * 256 * d + 4 * 64 * 256 + 5 * n, flops=2.0 * n * (256 * d + 64 * 256 + 64))
    if kind == "engine":
        layout, req, k = "paper", case["inst"], case["k"]
    else:
        layout, req, k = case["layout"], case.get("req", 0), case.get("k", 0)
    I, Q = case["inst"], len(LAYOUTS[layout][0])
    # an asked hash costs its 8 bytes and one 16-byte index slot, about half a request's hashes being needed
    match = req * (case.get("req_len", 0) / 2.0) * 0.6 * 24 + 8 * req
    select = I * (10 * case["blocks"] + Q * k * 8 + 4 * k)  # last_access, meta, offset; lists, scores, decision
    commit = I * k * (26 + 16 + 32 + 16)  # fields, index slot, recently_evicted entry and slot
    insert = I * k * (2 * 30 + 32)
    if kind == "match":
        return dict(bytes=match, flops=0)
    if kind == "select":
        return dict(bytes=select, flops=0)
    return dict(bytes=match + select + commit + insert, flops=0)


def tolerance(case):
    if case["kind"] == "predict":
        # fp32 sums of exact bf16 products: the path is 1.5e-7 to 4e-7 of the logits' norm from 64 bits
        # (another order of the sums may be as far off); a prediction may flip where |y| is that small
        return dict(rel=2e-6, differ=0.001)
    return "exact"  # ids, counts, and scores of a fixed fp32 recipe


# ------------------------------------------------------------------ 64-bit reference
def _exact_scores(pool, la, layout, now, k):
    """Per instance and queue the k smallest priorities (Eqs. 1-3; num_tokens in an evict-first queue)."""
    kinds, _, mu, sigma = LAYOUTS[layout]
    m = api.unpack_meta(pool.meta)
    off = pool.off.long() & 0xFFFFFFFF
    dt = (now - la.long()).clamp(min=0).double()
    out = torch.zeros((pool.n_inst, len(kinds), k), dtype=torch.float64, device="cuda")
    able = m["valid"] & m["leaf"] & ~m["ref"]
    for q, kind in enumerate(kinds):
        if kind == EF:
            key = m["ntok"].double()
        else:
            if kind == LN:
                p = 0.5 * torch.special.erfc((dt.clamp(min=1.0).log() - mu[q]) / (sigma[q] * math.sqrt(2.0)))
            elif kind == STRUCT:
                p = 1.0 - (off & 0xFFFF).double() / (off >> 16).double()
            else:
                p = torch.ones_like(dt)
            key = torch.where(dt > 0, p / dt.clamp(min=1.0), torch.full_like(dt, math.inf))
        mine = able & (m["queue"] == q)
        for i in range(pool.n_inst):
            sl = slice(i * pool.N, (i + 1) * pool.N)
            v = key[sl][mine[sl]]
            c = min(k, v.numel())
            if c:
                out[i, q, :c] = torch.topk(v, c, largest=False, sorted=True).values
    return [out[:, q] for q in range(len(kinds))]


def _touched(s):
    """last_access after the pass's prefix match: the leading cached hashes of every request."""
    pool = s["cache"].pool
    order = torch.argsort(pool.hash)
    keys = pool.hash[order]
    h = s["hashes"]
    at = torch.searchsorted(keys, h).clamp(max=keys.numel() - 1)
    block = order[at]
    inst = (s["inst"] if s["inst"] is not None else torch.zeros_like(s["lens"])).long()
    j = torch.arange(h.shape[1], device="cuda")[None, :]
    hit = (keys[at] == h) & (block // pool.N == inst[:, None]) & (j < s["lens"][:, None])
    hit = hit.long().cumprod(1).bool()
    la = pool.last_access.clone()
    la[block[hit]] = s["now"]
    return la


def exact(case, seed):
    kind = case["kind"]
    if kind in ("engine", "match"):
        return None  # whole numbers only
    s = prepare(case, seed)
    if kind == "predict":
        w = {n: (t.view(torch.bfloat16) if n == "w1" else t).double() for n, t in s["w"].items()}
        y = torch.relu(s["h"].view(torch.bfloat16).double() @ w["w1"].T + w["b1"])
        y = torch.relu(y @ w["w2"].T + w["b2"])
        return dict(logit=y @ w["w3"] + w["b3"], pred=None)
    pool = s["cache"].pool
    if kind == "select":
        return dict(scores=_exact_scores(pool, pool.last_access, case["layout"], s["now"] + 1, case["k"]))
    return dict(scores=_exact_scores(pool, _touched(s), case["layout"], s["now"], case["k"]))
