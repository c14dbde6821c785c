"""The calls whose speed matters to a program that serves vision-language models with this library.

Six paths, each through the public entry points of `paper_2606_03075_amd.binding`:

  evict         the whole eviction pass after a prefill, EvictionBuffers.evict: score, budget,
                vision scores, select, compact
  score         its scoring alone, in the default order: text statistics and text scores, layer
                budgets, vision scores of the layers whose budget reaches past the text
  score_lse     scoring from row normalisers that the prefill's attention kernel returned
  retain        what follows given scores: budgets, retained positions, compacted cache; contiguous,
                or with `page` the page table and the paged cache of a serving loop
  decode        one decode step over the pruned cache of a batch in lockstep
  decode_paged  one decode step of a continuous batch: every sequence at its own step, some slots
                idle, the cache in pages of a shared pool

Values follow the recipes of workloads/gen.py, drawn on the GPU: text keys and queries N(0, 1),
vision keys around a mean per KV head (a slowly moving mean per frame for video), token 0 an
attention sink, and with `gap` the depth profile of the text-to-vision attention, which spreads
the layers' budgets over an order of magnitude.
"""

import math

import numpy as np
import torch

from paper_2606_03075_amd import binding as bd

# Query heads, KV heads, head_dim of the model shapes in workloads/configs.py, and the grouped
# shapes of the tests.
_TINY = dict(hq=4, hkv=4, d=64)
_MHA32 = dict(hq=32, hkv=32, d=128)
_MHA40 = dict(hq=40, hkv=40, d=128)
_GQA7 = dict(hq=28, hkv=4, d=128)
_GQA4 = dict(hq=32, hkv=8, d=128)
_GQA8_64 = dict(hq=16, hkv=2, d=64)

_PLAIN = dict(frames=0, gap=0.0, head_mode=0, sink=0, recent=0, vision_only=False, reserve=64, page=0)


def _case(path, heads, batch, layers, sys, vis, qst, rho, **more):
    return dict(_PLAIN, path=path, batch=batch, layers=layers, sys=sys, vis=vis, qst=qst, rho=rho, **heads, **more)


def listed():
    cases = {
        # one layer of a small model, a prompt of 168 tokens: every kernel is a few workgroups
        "evict_tiny": _case("evict", _TINY, 1, 1, 8, 144, 16, 0.5),
        # one image question on a 7B model: the whole pass, as an interactive server calls it
        "evict_llava15": _case("evict", _MHA32, 1, 32, 35, 576, 40, 0.10),
        # a batch of multi-tile images on a 7B model: one long read of the keys per sweep
        "score_llavanext": _case("score", _MHA32, 4, 32, 35, 2880, 64, 0.05),
        # one video question on a grouped-query model: few units, long key rows
        "score_video_one": _case("score", _GQA7, 1, 28, 16, 8192, 48, 0.05, frames=16),
        # a batch of videos whose prefill kernel kept the text rows' log-sum-exp
        "score_lse_video": _case("score_lse", _GQA7, 8, 28, 16, 8192, 48, 0.05, frames=16),
        # 13B class, 16 sequences, long questions: the largest batch of the configurations
        "score_13b": _case("score", _MHA40, 16, 40, 35, 2880, 256, 0.10),
        # budgets, selection and compaction of the multi-tile batch, layers of very different budgets
        "retain_llavanext": _case("retain", _MHA32, 4, 32, 35, 2880, 64, 0.05, gap=6.0, reserve=128),
        # a video batch admitted into the paged pool of a serving loop
        "retain_video_paged": _case("retain", _GQA7, 8, 28, 16, 8192, 48, 0.10, gap=6.0, reserve=128, page=16),
        # the shortest decode step in use: one sequence, about 33 retained tokens a layer
        "decode_llava15": _case("decode", _MHA32, 1, 32, 35, 576, 40, 0.05),
        # the decode step of the multi-tile batch: a stream of 0.45 GB
        "decode_llavanext": _case("decode", _MHA32, 4, 32, 35, 2880, 64, 0.05, reserve=128),
        # one layer's decode attention, as a model's forward pass calls it between its projections
        "decode_layer_video": _case("decode", _GQA7, 8, 1, 16, 8192, 48, 0.10, reserve=128),
        # continuous batching over pages, grouped queries, sequences of different lengths
        "decode_paged_video": _case("decode_paged", _GQA7, 8, 28, 16, 8192, 48, 0.05, gap=6.0, reserve=128, page=16),
    }
    return [dict(c, name=n) for n, c in cases.items()]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    while True:
        path = rng.choice(["evict", "score", "score", "score_lse", "retain", "decode", "decode", "decode_paged"])
        heads = rng.choice([_TINY, _MHA32, _MHA32, _MHA40, _GQA7, _GQA7, _GQA4, _GQA8_64])
        small = heads in (_TINY, _GQA8_64)
        # a whole model, or one layer or a few of it (a pass per layer while the prefill runs)
        layers = rng.choice([1, _log(rng, 1, 40), rng.randint(16, 40), rng.randint(24, 40)])
        c = _case(path, heads, _log(rng, 1, 16), 1 if small and rng.random() < 0.3 else layers,
                  rng.randint(0, 100), _log(rng, 100, 9000), _log(rng, 8, 256), round(rng.uniform(0.04, 0.5), 3),
                  gap=rng.choice([0.0, 0.0, 6.0]), reserve=rng.choice([1, 32, 64, 128, 256]))
        if rng.random() < 0.3:
            c.update(sink=4, recent=1)
        if rng.random() < 0.2:
            c.update(vision_only=True)
        if rng.random() < 0.15:
            c.update(head_mode=1)
        if rng.random() < 0.3:
            frames = rng.choice([4, 8, 16])
            c.update(frames=frames, vis=max(c["vis"] // frames, 1) * frames)
        if path == "decode_paged" or (path == "retain" and rng.random() < 0.5):
            c.update(page=rng.choice([1, 16, 16, 32, 64, 128]))
            if -(-(_tokens(c) + c["reserve"]) // c["page"]) > 4096:
                continue
        if path == "evict" and c["batch"] * c["layers"] > 64:
            continue  # ranks that two correct sums order differently are rare in small batches only
        size = c["batch"] * c["layers"] * c["hkv"] * _tokens(c) * c["d"] * 2
        if size > 8e9 or work(c)["flops"] > 2e12 or work(c)["bytes"] > 16e9:
            continue
        return c


# ------------------------------------------------------------------------------------- shapes
def _tokens(c):
    return c["sys"] + c["vis"] + c["qst"]


def _problem(c):
    return bd.make_problem(c["batch"], c["layers"], c["hq"], c["hkv"], c["d"], c["sys"], c["vis"], c["qst"])


def _opts(c):
    return bd.make_opts(head_mode=c["head_mode"], n_sink=c["sink"], n_recent=c["recent"], vision_only=c["vision_only"])


def _forced_vision(c):
    n, fs = _tokens(c), min(c["sink"], _tokens(c))
    forced = set(range(fs)) | set(range(max(n - c["recent"], fs), n))
    return sum(1 for p in forced if c["sys"] <= p < c["sys"] + c["vis"])


def _total(c):
    """The budget given to tgvkv_budget: a share of all cached tokens, or of the vision tokens."""
    if c["vision_only"]:
        return int(math.floor(c["rho"] * (c["vis"] - _forced_vision(c)) * c["layers"] + 0.5))
    return int(math.floor(c["rho"] * _tokens(c) * c["layers"] + 0.5))


def _kept(c):
    """Tokens a sequence keeps over its layers."""
    if c["vision_only"]:
        return _total(c) + c["layers"] * (c["sys"] + c["qst"] + _forced_vision(c))
    return _total(c)


def work(case):
    c = case
    n, nt, d, bl = _tokens(c), c["sys"] + c["qst"], c["d"], c["batch"] * c["layers"]
    g = 1 if c["head_mode"] == 0 else c["hkv"]
    kept = c["batch"] * _kept(c)
    keys = bl * c["hkv"] * n * d * 2
    queries = bl * c["hq"] * nt * d * 2
    scores = 4 * bl * (c["hq"] * nt + g * (2 * nt + c["vis"]) + 1)
    moved = 2 * 2 * kept * c["hkv"] * d * 2 + 4 * g * kept + 20 * bl
    visible = c["qst"] * (c["sys"] + c["vis"]) + c["qst"] * (c["qst"] + 1) // 2 + c["sys"] * (c["sys"] + 1) // 2
    flops = 2 * d * bl * c["hq"] * visible
    if c["path"] == "evict":
        return {"bytes": keys + queries + scores + moved, "flops": flops}
    if c["path"] in ("score", "score_lse"):
        return {"bytes": keys + queries + scores, "flops": flops}
    if c["path"] == "retain":
        return {"bytes": moved + 4 * bl * (g * (nt + c["vis"]) + 1), "flops": 0}
    step = _step(c)
    rows = kept + bl * (step + 1)
    return {"bytes": 2 * rows * c["hkv"] * d * 2 + bl * c["hq"] * d * (2 + 4) + 2 * bl * c["hkv"] * d * 2,
            "flops": 4 * d * rows * c["hq"]}


def _step(c):
    return c["reserve"] // 2


# ------------------------------------------------------------------------------------- inputs
def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed))
    return g


def _randn(g, *shape, dtype=torch.bfloat16):
    return torch.randn(*shape, generator=g, device="cuda", dtype=dtype)


def _means(c, g, frames):
    """Mean vision keys [B, L, hkv, frames, d]: an AR(1) walk over the frames."""
    eps = _randn(g, c["batch"], c["layers"], c["hkv"], frames, c["d"], dtype=torch.float32)
    for f in range(1, frames):
        eps[..., f, :] = math.sqrt(0.99) * eps[..., f - 1, :] + 0.1 * eps[..., f, :]
    return eps


def _depth(c, g):
    """Shift of the question rows' vision logits per (sequence, layer), as gen.vision_logit_shift."""
    x = torch.arange(c["layers"], device="cuda", dtype=torch.float32) / max(c["layers"] - 1, 1)
    z = _randn(g, c["batch"], c["layers"], dtype=torch.float32)
    return -c["gap"] * (1.0 - 0.85 * torch.exp(-x / 0.08) - 0.25 * x) + 0.5 * z


def _prefill(c, seed, values=False):
    """q_text [B, L, hq, N_t, d], k (and v) [B, L, hkv, N, d] of one prefill."""
    g = _gen(seed)
    b, l, n, s, d = c["batch"], c["layers"], _tokens(c), c["sys"], c["d"]
    frames = max(c["frames"], 1)
    mu = _means(c, g, frames)
    q = _randn(g, b, l, c["hq"], s + c["qst"], d)
    if c["gap"] > 0:
        m = mu.mean(dim=3)
        shift = _depth(c, g)[:, :, None, None] * math.sqrt(d) / (m * m).sum(-1, keepdim=True) * m
        shift = shift.repeat_interleave(c["hq"] // c["hkv"], dim=2)[:, :, :, None, :]
        q[:, :, :, s:] = (q[:, :, :, s:].float() + shift).to(torch.bfloat16)
    k = torch.empty(b, l, c["hkv"], n, d, dtype=torch.bfloat16, device="cuda")
    sigma = 0.25 if c["frames"] == 0 else 0.3
    for i in range(b):
        k[i] = _randn(g, l, c["hkv"], n, d)
        part = k[i, :, :, s:s + c["vis"]].unflatten(2, (frames, -1))
        part.mul_(sigma).add_(mu[i][:, :, :, None, :].to(torch.bfloat16))
    k[:, :, :, 0] *= 4
    return (q, k, _randn(g, b, l, c["hkv"], n, d)) if values else (q, k)


def _normalisers(c, q, k, dtype=torch.float32, to=None):
    """Natural log-sum-exp of every text row, [B, L, hq, N_t]: what a prefill attention kernel returns."""
    out = []
    for i in range(c["batch"]):
        for j in range(c["layers"]):
            out.append(torch.logsumexp(_logits(c, q[i, j], k[i, j], dtype), dim=-1))
    return torch.stack(out).view(c["batch"], c["layers"], c["hq"], -1).to(to or dtype)


def _hidden(c):
    """[N_t, N]: keys that a text row does not see."""
    n, s = _tokens(c), c["sys"]
    pos = torch.arange(n, device="cuda")
    text = torch.cat([pos[:s], pos[s + c["vis"]:]])
    return pos[None, :] > text[:, None]


def _logits(c, q, k, dtype):
    """[hq, N_t, N] masked logits of one (sequence, layer)."""
    kk = k.to(dtype).repeat_interleave(c["hq"] // c["hkv"], dim=0).transpose(1, 2).contiguous()
    z = torch.matmul(q.to(dtype), kk).mul_(1.0 / math.sqrt(c["d"]))
    return z.masked_fill_(_hidden(c), float("-inf"))


def _masses(c, g):
    """Layers' text-to-vision masses [B, L]: what scoring finds for these inputs, roughly."""
    logit = _depth(c, g) if c["gap"] > 0 else 0.02 * _randn(g, c["batch"], c["layers"], dtype=torch.float32)
    odds = torch.exp(logit) * (c["vis"] / max(c["sys"] + c["qst"], 1)) * 0.3
    return (c["qst"] * odds / (1 + odds)).contiguous()


def _drawn_budgets(c, g):
    """Layer budgets [B][L] in proportion to drawn masses, whole numbers that sum to the kept tokens."""
    m = _masses(c, g).double().cpu().numpy()
    always, cap = (c["sys"] + c["qst"] + _forced_vision(c), c["vis"] - _forced_vision(c)) if c["vision_only"] else (0, _tokens(c))
    out = []
    for row in m:
        share, left = np.zeros(c["layers"]), float(_total(c))
        open_ = np.ones(c["layers"], bool)
        while left > 0 and open_.any():
            x = left * row[open_] / row[open_].sum()
            share[open_] = x
            over = open_ & (share > cap)
            if not over.any():
                break
            share[over] = cap
            open_ &= ~over
            left = _total(c) - cap * float((~open_).sum())
        b = np.floor(share).astype(np.int64)
        order = np.argsort(-(share - b) + (b >= cap), kind="stable")
        b[order[:_total(c) - int(b.sum())]] += 1
        out.append(b + always)
    return np.stack(out).astype(np.int32)


def _order(b):
    """Longest segments first, as tgvkv_budget's unit_order."""
    layers, batch = b.shape[1], b.shape[0]
    o = np.empty((layers, batch), np.int32)
    for i in range(batch):
        o[:, i] = i * layers + np.argsort(-b[i].astype(np.int64), kind="stable")
    return torch.from_numpy(o.reshape(-1)).cuda()


def _new_token(c, g):
    return [_randn(g, c["batch"], c["layers"], h, c["d"]) for h in (c["hq"], c["hkv"], c["hkv"])]


def _cache(c, seed):
    """The pruned cache of a batch in lockstep, every slot filled, and the step's token."""
    g = _gen(seed)
    b = _drawn_budgets(c, g)
    rows = int(b.sum()) + b.size * c["reserve"]
    kc, vc = (_randn(g, rows * c["hkv"] * c["d"]) for _ in range(2))
    return b, kc, vc, _new_token(c, g)


def _paged(c, seed):
    """A pool in use: the batch's pages scattered over it, one slot in eight idle."""
    g = _gen(seed)
    b = _drawn_budgets(c, g)
    r = np.random.default_rng(int(seed))
    steps = r.integers(0, c["reserve"], c["batch"]).astype(np.int32)
    if c["batch"] >= 4:
        steps[r.random(c["batch"]) < 0.125] = -1
    need = -(-(b.astype(np.int64) + c["reserve"]) // c["page"])
    width, n_pages = bd.page_plan(_problem(c), _opts(c), _total(c), c["reserve"], c["page"])
    pool = [_randn(g, n_pages, c["hkv"], c["page"], c["d"]) for _ in range(2)]
    ids = r.permutation(n_pages).astype(np.int32)
    table = np.full((b.size, width), -1, np.int32)
    at = 0
    for i, n in enumerate(need.reshape(-1)):
        table[i, :n] = ids[at:at + n]
        at += n
    return b, steps, table, pool, _new_token(c, g)


def prepare(case, seed):
    c = case
    p, o = _problem(c), _opts(c)
    st = {"path": c["path"], "problem": p, "opts": o}
    if c["path"] in ("evict", "score", "score_lse"):
        t = _prefill(c, seed, values=c["path"] == "evict")
        buf = bd.EvictionBuffers(p, o, _total(c), c["reserve"])
        if c["path"] == "evict":
            buf.kc.zero_()
            buf.vc.zero_()
        elif c["path"] == "score_lse":
            buf.lse.copy_(_normalisers(c, *t))
        st.update(buf=buf, inputs=t)
    elif c["path"] == "retain":
        g = _gen(seed)
        n = _tokens(c)
        buf = bd.EvictionBuffers(p, o, _total(c), c["reserve"])
        buf.kc.zero_()
        buf.vc.zero_()
        buf.tv_mass.copy_(_masses(c, g))
        # head means of attention: log-normal over the tokens
        buf.s_vis.copy_(torch.exp(0.5 * _randn(g, *buf.s_vis.shape, dtype=torch.float32)) / n)
        buf.s_txt.copy_(torch.exp(_randn(g, *buf.s_txt.shape, dtype=torch.float32)))
        k, v = (_randn(g, c["batch"], c["layers"], c["hkv"], n, c["d"]) for _ in range(2))
        st.update(buf=buf, inputs=(k, v), page=c["page"])
        if c["page"]:
            width, pages = bd.page_plan(p, o, _total(c), c["reserve"], c["page"])
            r = np.random.default_rng(int(seed))
            st.update(free=torch.from_numpy(r.permutation(pages).astype(np.int32)).cuda(),
                      table=torch.empty(c["batch"] * c["layers"], width, dtype=torch.int32, device="cuda"),
                      used=torch.zeros(1, dtype=torch.int64, device="cuda"),
                      pool=[torch.zeros(pages, c["hkv"], c["page"], c["d"], dtype=torch.bfloat16, device="cuda")
                            for _ in range(2)])
    elif c["path"] == "decode":
        b, kc, vc, new = _cache(c, seed)
        buf = bd.EvictionBuffers(p, o, _total(c), c["reserve"])
        buf.kc, buf.vc = kc, vc
        buf.budgets.copy_(torch.from_numpy(b))
        seg = np.concatenate([[0], np.cumsum(b.reshape(-1).astype(np.int64) + c["reserve"])])
        buf.seg_offsets.copy_(torch.from_numpy(seg))
        buf.unit_order = _order(b)
        st.update(buf=buf, new=new, step=_step(c))
    else:
        b, steps, table, pool, new = _paged(c, seed)
        pages = bd.PagedPool(c["hkv"], c["d"], c["page"], 1)
        pages.k_pool, pages.v_pool = pool
        ws = bd.workspace_size(p, o, bd.CALL_DECODE)
        st.update(pages=pages, budgets=torch.from_numpy(b).cuda(), steps=torch.from_numpy(steps).cuda(),
                  table=torch.from_numpy(table).cuda(), order=_order(b), new=new, reserve=c["reserve"],
                  out=torch.zeros(c["batch"], c["layers"], c["hq"], c["d"], device="cuda"),
                  ws=torch.empty(max(1, ws), dtype=torch.uint8, device="cuda"))
    return st


# ------------------------------------------------------------------------------------- a pass
def run(state):
    st = state
    if st["path"] == "evict":
        buf = st["buf"]
        buf.evict(*st["inputs"])
        return {"lse": buf.lse, "s_txt": buf.s_txt, "w_txt": buf.w_txt, "tv_mass": buf.tv_mass, "s_vis": buf.s_vis,
                "budgets": buf.budgets, "idx": buf.idx, "kc": buf.kc, "vc": buf.vc}
    if st["path"] == "score":
        buf, (q, k) = st["buf"], st["inputs"]
        buf.score(q, k, bd.SCORE_STATS | bd.SCORE_TEXT)
        buf.budget()
        buf.score(q, k, bd.SCORE_VISION, budgets=buf.budgets)
        return {"lse": buf.lse, "s_txt": buf.s_txt, "w_txt": buf.w_txt, "tv_mass": buf.tv_mass, "s_vis": buf.s_vis,
                "budgets": buf.budgets}
    if st["path"] == "score_lse":
        buf, (q, k) = st["buf"], st["inputs"]
        buf.score(q, k, bd.SCORE_TEXT | bd.SCORE_VISION | bd.SCORE_LSE_IN)
        return {"s_txt": buf.s_txt, "w_txt": buf.w_txt, "tv_mass": buf.tv_mass, "s_vis": buf.s_vis}
    if st["path"] == "retain":
        buf, (k, v) = st["buf"], st["inputs"]
        buf.budget()
        buf.select()
        out = {"budgets": buf.budgets, "idx": buf.idx, "idx_offsets": buf.idx_offsets, "seg_offsets": buf.seg_offsets,
               "unit_order": buf.unit_order}
        if not st["page"]:
            buf.compact(k, v)
            return dict(out, kc=buf.kc, vc=buf.vc)
        p, o = st["problem"], st["opts"]
        bd.tgvkv_page_table(p, o, buf.budgets, buf.total_budget, buf.decode_reserve, st["page"], st["free"], st["table"],
                            st["used"])
        bd.tgvkv_compact_paged(p, o, k, v, buf.idx, buf.budgets, buf.idx_offsets, buf.total_budget, st["table"],
                               st["page"], *st["pool"], unit_order=buf.unit_order)
        return dict(out, table=st["table"], used=st["used"], k_pool=st["pool"][0], v_pool=st["pool"][1])
    if st["path"] == "decode":
        buf = st["buf"]
        return {"out": buf.decode(st["step"], *st["new"]), "kc": buf.kc, "vc": buf.vc}
    pages = st["pages"]
    out = pages.decode(st["problem"], st["opts"], st["table"], st["budgets"], st["reserve"], st["steps"], *st["new"],
                       st["out"], st["ws"], unit_order=st["order"])
    return {"out": out, "k_pool": pages.k_pool, "v_pool": pages.v_pool}


# ------------------------------------------------------------------------------------- how close
def tolerance(case):
    if case["path"] == "retain":
        return "exact"
    # 32-bit sums of 16-bit inputs.  Measured against 64 bits: scores within 4e-7 (2-norm), decode
    # within 1.6e-7 for plain heads and 1.6e-6 for grouped ones, whose probabilities enter the
    # product with the values with about 16 significant bits.
    if case["path"] in ("decode", "decode_paged"):
        return {"rel": 8e-6, "max": 8e-5}
    return {"rel": 4e-6, "max": 4e-5}


def exact(case, seed):
    c = case
    if c["path"] == "retain":
        return None
    if c["path"] in ("decode", "decode_paged"):
        return _exact_decode(c, seed)
    t = _prefill(c, seed)
    lse = _normalisers(c, *t, to=torch.float32).double() if c["path"] == "score_lse" else None
    got = {n: [] for n in ("lse", "s_txt", "w_txt", "tv_mass", "s_vis")}
    groups = 1 if c["head_mode"] == 0 else c["hkv"]
    nt, s = c["sys"] + c["qst"], c["sys"]
    for i in range(c["batch"]):
        for j in range(c["layers"]):
            z = _logits(c, t[0][i, j], t[1][i, j], torch.float64)
            row = torch.logsumexp(z, dim=-1) if lse is None else lse[i, j]
            a = z.sub_(row[..., None]).exp_()
            got["lse"].append(row)
            a = a.unflatten(0, (groups, -1)).mean(1)  # [groups, N_t, N]
            vis = a[:, :, s:s + c["vis"]]
            s_txt = torch.cat([a[:, :, :s], a[:, :, s + c["vis"]:]], dim=2).sum(1)
            w = s_txt / torch.arange(nt, 0, -1, device="cuda", dtype=torch.float64)
            w = w / w.sum(-1, keepdim=True)
            got["s_txt"].append(s_txt)
            got["w_txt"].append(w)
            got["tv_mass"].append(vis.sum((1, 2)).mean())
            got["s_vis"].append((w[:, :, None] * vis).sum(1))
    shape = (c["batch"], c["layers"])
    out = {n: torch.stack(v).view(*shape, *v[0].shape) for n, v in got.items()}
    if c["path"] == "score_lse":
        out.pop("lse")
        return out
    # layers whose budget ends within the text get no vision scores: where the masses leave that
    # open, the vision scores of the batch have no value here
    m = out["tv_mass"]
    least = (_total(c) * m / m.sum(1, keepdim=True)).min().item()
    if least <= (0 if c["vision_only"] else nt + _forced_vision(c) + c["sink"] + c["recent"]) + 2:
        out["s_vis"] = None
    out["budgets"] = None
    if c["path"] == "evict":
        out.update(idx=None, kc=None, vc=None)
    return out


def _attend(c, q, k, v):
    """[hq, d] in 64 bits; q [hq, d], k and v [hkv, n, d]."""
    q = q.double().unflatten(0, (c["hkv"], -1))
    p = torch.softmax(torch.matmul(q, k.double().transpose(1, 2).contiguous()) / math.sqrt(c["d"]), dim=-1)
    return torch.matmul(p, v.double()).flatten(0, 1)


def _exact_decode(c, seed):
    out = torch.zeros(c["batch"], c["layers"], c["hq"], c["d"], dtype=torch.float64, device="cuda")
    if c["path"] == "decode":
        b, kc, vc, (q, kn, vn) = _cache(c, seed)
        at, step = 0, _step(c)
        for i in range(c["batch"]):
            for j in range(c["layers"]):
                cap = int(b[i, j]) + c["reserve"]
                k, v = (x[at * c["hkv"] * c["d"]:(at + cap) * c["hkv"] * c["d"]].view(c["hkv"], cap, c["d"])
                        for x in (kc, vc))
                k[:, int(b[i, j]) + step], v[:, int(b[i, j]) + step] = kn[i, j], vn[i, j]
                n = int(b[i, j]) + step + 1
                out[i, j] = _attend(c, q[i, j], k[:, :n], v[:, :n])
                at += cap
        return {"out": out, "kc": kc.double(), "vc": vc.double()}
    b, steps, table, (kp, vp), (q, kn, vn) = _paged(c, seed)
    for i in range(c["batch"]):
        for j in range(c["layers"]):
            if steps[i] < 0:
                continue
            last = int(b[i, j]) + int(steps[i])
            ids = torch.from_numpy(table[i * c["layers"] + j, :last // c["page"] + 1].astype(np.int64)).cuda()
            kp[ids[-1], :, last % c["page"]], vp[ids[-1], :, last % c["page"]] = kn[i, j], vn[i, j]
            k, v = (x[ids].transpose(0, 1).flatten(1, 2)[:, :last + 1] for x in (kp, vp))
            out[i, j] = _attend(c, q[i, j], k, v)
    return {"out": out, "k_pool": kp.double(), "v_pool": vp.double()}
