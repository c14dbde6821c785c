"""Launch plans away from the benchmark's shapes: each test runs a plan at the sizes where it changes, against the oracle.

Scores are held to 2e-5 of the 64-bit oracle: logits up to 20 in base 2, rounded in 32 bits, move an exponential by about
2e-6, and the sums of positive terms, in partial sums of a few hundred terms, as much again.  One key left out or
counted twice at the edge of a share or a ragged tile shows (test_ranges_cpu.py): it moves the normaliser of some row by
more than that."""

import numpy as np
import pytest

import oracle.tgvkv_oracle as O
from paper_2606_03075_amd import binding as bd
from tests.gpu_util import assert_close_rel, dev_bf16, host, log, oracle_scores
from workloads import make_prefill_tensors
from workloads.configs import custom_config

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def lib():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    return bd.load_library()


SCORE_BOUND = 2e-5  # absolute for the normalisers (natural log), relative for the scores


def check_scores(cfg, head_mode=0, phase_lists=((bd.SCORE_ALL,),)):
    """Scores of every (sequence, layer) against the oracle, for each way of asking for the phases."""
    import torch
    t = make_prefill_tensors(cfg, seed=5, names=("q_text", "k"))
    ref = [[oracle_scores(t["q_text"][b, l], t["k"][b, l], cfg, head_mode) for l in range(cfg.layers)]
           for b in range(cfg.batch)]
    q, k = dev_bf16(t["q_text"]), dev_bf16(t["k"])
    for phases in phase_lists:
        buf = bd.EvictionBuffers(bd.problem_from(cfg), bd.make_opts(head_mode=head_mode), 0, 1)
        for ph in phases:
            if ph & bd.SCORE_LSE_IN:
                lse = np.stack([[r["lse"] for r in row] for row in ref]).astype(np.float32)
                buf.lse.copy_(torch.from_numpy(lse))
            buf.score(q, k, ph)
        torch.cuda.synchronize()
        for b in range(cfg.batch):
            for l in range(cfg.layers):
                r = ref[b][l]
                assert_close_rel("lse", host(buf.lse[b, l]), r["lse"], rtol=0.0, atol=SCORE_BOUND)
                for n in ("s_txt", "w_txt", "tv_mass", "s_vis"):
                    assert_close_rel(n, host(getattr(buf, n)[b, l]), r[n], rtol=SCORE_BOUND)


SPLIT_STATS = {
    # 12 and 11 key tiles of one row slot per wave: the shortest sweep in shares and the longest whole one
    "short_12_tiles": dict(heads_q=4, heads_kv=4, n_sys=5, n_vis=690, n_qst=50),
    "whole_11_tiles": dict(heads_q=4, heads_kv=4, n_sys=5, n_vis=650, n_qst=49),
    # 21 row blocks, six slots: two shares, the last tile a single key
    "gqa7_last_key": dict(heads_q=14, heads_kv=2, n_sys=17, n_vis=704, n_qst=48),
    # two key parts: a last share of one tile, its last key alone in a 16-key block
    "key_parts": dict(heads_q=2, heads_kv=2, n_sys=7, n_vis=800, n_qst=26),
    # shares that hold no vision key, or nothing but masked question keys for the early rows
    "question_shares": dict(heads_q=2, heads_kv=2, n_sys=130, n_vis=70, n_qst=700),
    "system_shares": dict(heads_q=2, heads_kv=2, n_sys=700, n_vis=70, n_qst=20),
    # several row groups per unit, each in shares; the text pass per query head in chunks of key blocks
    "row_groups": dict(heads_q=16, heads_kv=1, n_sys=40, n_vis=900, n_qst=160),
    # text rows that do not fit the staged text pass
    "long_text_split": dict(heads_q=2, heads_kv=1, n_sys=10, n_vis=100, n_qst=4000, layers=1),
    # many shares, and head_dim 64 with no system text
    "many_shares": dict(heads_q=3, heads_kv=1, n_sys=9, n_vis=8300, n_qst=33),
    "d64": dict(heads_q=8, heads_kv=2, head_dim=64, n_sys=0, n_vis=900, n_qst=19),
}


@pytest.mark.parametrize("name", sorted(SPLIT_STATS))
def test_split_statistics(lib, name):
    """The statistics sweep in shares of the keys: with workgroups of their own, merged by the text pass (both phases in
    one call) and by the merge kernel (statistics alone, then text)."""
    log(f"split statistics {name}")
    cfg = custom_config(name=name, **dict(dict(batch=1, layers=2), **SPLIT_STATS[name]))
    check_scores(cfg, 0, ((bd.SCORE_ALL,), (bd.SCORE_STATS, bd.SCORE_TEXT, bd.SCORE_VISION)))


SPLIT_VISION = {
    # shares of a few tiles, the last one ragged; shares of a row plan with its own vision launch shape; two row groups
    "mha": dict(heads_q=4, heads_kv=4, n_sys=5, n_vis=1201, n_qst=50),
    "three_blocks": dict(heads_q=4, heads_kv=4, n_sys=0, n_vis=449, n_qst=40),
    "below_a_share": dict(heads_q=4, heads_kv=4, n_sys=3, n_vis=190, n_qst=20),
    "gqa7_d64": dict(heads_q=14, heads_kv=2, head_dim=64, n_sys=3, n_vis=700, n_qst=50),
    "most_shares": dict(heads_q=7, heads_kv=1, n_sys=16, n_vis=6500, n_qst=48),
    "no_vision": dict(heads_q=4, heads_kv=2, n_sys=30, n_vis=0, n_qst=20),
    "no_question": dict(heads_q=4, heads_kv=2, n_sys=30, n_vis=300, n_qst=0),
}


@pytest.mark.parametrize("name", sorted(SPLIT_VISION))
def test_split_vision(lib, name):
    """The vision sweep's keys split over workgroups, and with given normalisers the layers' masses from the shares'
    row masses."""
    log(f"split vision {name}")
    cfg = custom_config(name=name, **dict(dict(batch=1, layers=2), **SPLIT_VISION[name]))
    check_scores(cfg, 0, ((bd.SCORE_ALL,), (bd.SCORE_TEXT | bd.SCORE_VISION | bd.SCORE_LSE_IN,)))


# 16-row blocks per KV head, (query heads, question rows): the edges of every slot count and of the row groups
ROW_PLANS = {5: (5, 16), 8: (4, 30), 9: (3, 48), 12: (4, 33), 13: (13, 9), 16: (16, 16), 17: (1, 260), 20: (4, 80),
             21: (7, 48), 24: (12, 20), 25: (5, 75), 28: (7, 64), 33: (11, 48), 49: (7, 100)}


@pytest.mark.parametrize("head_dim", [64, 128])
@pytest.mark.parametrize("blocks", sorted(ROW_PLANS))
def test_row_plans(lib, blocks, head_dim):
    """Question rows dealt over row groups and row slots, statistics and vision sweep, with and without given
    normalisers (whose sweep also sums each row)."""
    heads, nq = ROW_PLANS[blocks]
    assert heads * ((nq + 15) // 16) == blocks
    log(f"row plan {blocks} blocks d{head_dim}")
    cfg = custom_config(name=f"nb{blocks}", batch=1, layers=1, heads_q=2 * heads, heads_kv=2, head_dim=head_dim, n_sys=7,
                        n_vis=150, n_qst=nq)
    check_scores(cfg, 1, ((bd.SCORE_ALL,), (bd.SCORE_TEXT | bd.SCORE_VISION | bd.SCORE_LSE_IN,)))


def test_one_order_in_any_batch(lib):
    """With ONE_ORDER a sequence's scores are the same bits alone and in a batch; with given normalisers the flag is
    refused."""
    import torch
    log("one order")
    shape = dict(layers=3, heads_q=14, heads_kv=2, n_sys=9, n_vis=900, n_qst=60)
    t = make_prefill_tensors(custom_config(batch=80, **shape), seed=2, names=("q_text", "k"), seqs=range(2))
    q, k = (dev_bf16(t[n]).repeat(40, 1, 1, 1, 1) for n in ("q_text", "k"))

    def scores(batch):
        buf = bd.EvictionBuffers(bd.problem_from(custom_config(batch=batch, **shape)), None, 0, 1)
        buf.score(q[:batch].contiguous(), k[:batch].contiguous(), bd.SCORE_ALL | bd.SCORE_ONE_ORDER)
        return buf
    one, many = scores(1), scores(80)
    for n in ("lse", "s_txt", "w_txt", "tv_mass", "s_vis"):
        a, b = getattr(one, n), getattr(many, n)
        assert torch.equal(a[0], b[0]) and torch.equal(b[0], b[78]) and torch.equal(b[1], b[79]), n
    with pytest.raises(bd.TgvkvError):
        one.score(q[:1], k[:1], bd.SCORE_TEXT | bd.SCORE_VISION | bd.SCORE_LSE_IN | bd.SCORE_ONE_ORDER)


# one sequence of each row plan: its key parts, slots and row groups, text passes staged whole, in chunks and not at all
SEQUENCES = {
    "one_block": dict(heads_q=2, heads_kv=2, n_sys=35, n_vis=1501, n_qst=16),
    "two_blocks": dict(heads_q=2, heads_kv=2, n_sys=0, n_vis=2002, n_qst=30),
    "three_blocks_d64": dict(heads_q=2, heads_kv=2, head_dim=64, n_sys=70, n_vis=1700, n_qst=45),
    "one_slot": dict(heads_q=2, heads_kv=2, n_sys=130, n_vis=1500, n_qst=64),
    "two_slots": dict(heads_q=4, heads_kv=2, n_sys=9, n_vis=1333, n_qst=50),
    "three_slots": dict(heads_q=2, heads_kv=2, n_sys=20, n_vis=1100, n_qst=180),
    "four_slots_d64": dict(heads_q=8, heads_kv=2, head_dim=64, n_sys=20, n_vis=1100, n_qst=60),
    "five_slots": dict(heads_q=10, heads_kv=2, n_sys=5, n_vis=1250, n_qst=60),
    "six_slots": dict(heads_q=14, heads_kv=2, n_sys=16, n_vis=1300, n_qst=40),
    "six_slots_d64": dict(heads_q=14, heads_kv=2, head_dim=64, n_sys=100, n_vis=1300, n_qst=48),
    "row_groups": dict(heads_q=14, heads_kv=2, n_sys=3, n_vis=1100, n_qst=60),
    "long_text": dict(heads_q=14, heads_kv=2, n_sys=260, n_vis=700, n_qst=160),
    "unstaged_text": dict(heads_q=4, heads_kv=2, n_sys=3000, n_vis=600, n_qst=30),
    "short": dict(heads_q=4, heads_kv=2, n_sys=5, n_vis=300, n_qst=20),
}


@pytest.mark.parametrize("name", sorted(SEQUENCES))
def test_same_bits_in_any_batch(lib, name):
    """A sequence's scores are the same bits in a batch of any size, however the call is made: alone, where its keys are
    spread over workgroups, and where a workgroup takes a unit's keys whole, with more units than get a text workgroup
    per query head.  With given normalisers the layers' masses are sums over the batch's shares, and may differ."""
    import torch
    log(f"same bits in any batch {name}")
    shape = dict(dict(layers=1), **SEQUENCES[name])
    t = make_prefill_tensors(custom_config(batch=2, **shape), seed=2, names=("q_text", "k"))
    q, k = (dev_bf16(t[n]) for n in ("q_text", "k"))
    lse = torch.randn(2, 1, shape["heads_q"], shape["n_sys"] + shape["n_qst"], device="cuda").abs() + 7
    names = ("lse", "s_txt", "w_txt", "tv_mass", "s_vis")
    ways = {"all": (bd.SCORE_ALL,), "two": (bd.SCORE_STATS | bd.SCORE_TEXT, bd.SCORE_VISION),
            "phases": (bd.SCORE_STATS, bd.SCORE_TEXT, bd.SCORE_VISION), "one order": (bd.SCORE_ALL | bd.SCORE_ONE_ORDER,),
            "lse": (bd.SCORE_TEXT | bd.SCORE_VISION | bd.SCORE_LSE_IN,)}
    for way, phases in ways.items():
        first = None
        for batch in (1, 2, 40, 100, 150, 200, 260):
            order = torch.arange(batch, device="cuda") % 2
            buf = bd.EvictionBuffers(bd.problem_from(custom_config(batch=batch, **shape)), None, 0, 1)
            buf.ws_score.fill_(255)
            buf.lse.copy_(lse[order])
            for ph in phases:
                buf.score(q[order].contiguous(), k[order].contiguous(), ph)
            got = {n: getattr(buf, n).clone() for n in names if not (way == "lse" and n == "tv_mass")}
            if batch == 2:
                first = got
            elif batch == 1:
                alone = got
            for n, x in got.items():
                assert torch.isfinite(x).all(), (way, batch, n)
                assert torch.equal(x[0], alone[n][0]), (way, batch, n)
                assert first is None or torch.equal(x, first[n][order]), (way, batch, n)


# positions per row: each count of waves and register groups to its last position, the first past it, and past them all
SELECT_ROWS = [1, 65, 256, 257, 512, 768, 769, 1024, 1025, 1536, 3072, 3073, 4096, 4097, 6144, 9216, 9217, 12288, 12289]
SELECT_VALUES = {
    "spread": lambda r, n: r.standard_normal(n) * 10.0 ** r.uniform(-30, 30, n),   # the first digit settles little
    "close": lambda r, n: 1.0 + r.random(n) * 2.0 ** -12,                          # keys differ in the last 11 bits
    "tied": lambda r, n: r.integers(0, 3, n) - 1.0,                                # -1, 0 and 1: ties in the hundreds
    "equal": lambda r, n: np.full(n, 0.25),
    "outlier": lambda r, n: np.where(r.random(n) < 0.01, np.inf, np.where(r.random(n) < 0.01, -np.inf, r.random(n))),
}


@pytest.mark.parametrize("values", sorted(SELECT_VALUES))
@pytest.mark.parametrize("n", SELECT_ROWS)
def test_select_rows(lib, n, values):
    """The k-th largest by radix passes in registers (and, past them, from memory) and the ordered emission, against
    the oracle: whole numbers, so exact."""
    import torch
    log(f"select {n} {values}")
    r = np.random.default_rng(n)
    ns, nq = (3, 5) if n > 8 else (0, 0)
    nv, nt, layers = n - ns - nq, ns + nq, 9
    sv = SELECT_VALUES[values](r, layers * nv).astype(np.float32).reshape(1, layers, 1, nv)
    st = SELECT_VALUES[values](r, layers * nt).astype(np.float32).reshape(1, layers, 1, nt)
    bud = np.clip([0, 1, nt, nt + 1, nt + 2, nt + nv // 17, nt + nv // 2, n - 1, n], 0, n).reshape(1, layers)
    offsets = O.flat_offsets(bud.reshape(-1))
    for joint in (False, True):
        idx = torch.full((max(1, int(offsets[-1])),), -1, dtype=torch.int32, device="cuda")
        bd.tgvkv_select(bd.make_problem(1, layers, 2, 2, 64, ns, nv, nq), bd.make_opts(vision_rank=1, joint_rank=joint),
                        torch.from_numpy(sv).cuda(), torch.from_numpy(st).cuda() if nt else torch.zeros(1, device="cuda"),
                        torch.from_numpy(bud.astype(np.int32)).cuda(), torch.from_numpy(offsets).cuda(), idx)
        got = host(idx)
        for l in range(layers):
            args = (sv[0, l, 0].astype(np.float64), st[0, l, 0].astype(np.float64), int(bud[0, l]), ns, nv, nq)
            want = O.joint_select(*args, vis_scale=1.0) if joint else O.tpr_select(*args)
            assert np.array_equal(got[offsets[l]:offsets[l + 1]], want), (l, joint)


@pytest.mark.parametrize("n", [65, 769, 3073, 12288, 12289])
def test_select_all_ones_scores(lib, n):
    """Scores whose bits are all ones (a NaN, as in memory filled with 0xFF) are outside the contract, but they stay
    candidates: below every number, the lower position first, every retained position written and in range."""
    import torch
    log(f"select all-ones scores {n}")
    r = np.random.default_rng(n)
    ns, nq, nv = 3, 5, n - 8
    sv = r.standard_normal(nv).astype(np.float32)
    number = r.random(nv) < 0.3
    sv.view(np.uint32)[~number] = 0xFFFFFFFF
    st = r.standard_normal(ns + nq).astype(np.float32)
    few = int(number.sum())
    bud = np.array([8 + few // 2, 8 + few, 9 + few, 8 + (few + nv) // 2, n - 1, n], np.int32)
    offsets = O.flat_offsets(bud)
    layers = len(bud)
    idx = torch.full((int(offsets[-1]) + 64,), -1, dtype=torch.int32, device="cuda")
    rows = [torch.from_numpy(np.broadcast_to(x, (1, layers, 1, x.size)).copy()).cuda() for x in (sv, st)]
    bd.tgvkv_select(bd.make_problem(1, layers, 2, 2, 64, ns, nv, nq), None, *rows,
                    torch.from_numpy(bud.reshape(1, layers)).cuda(), torch.from_numpy(offsets).cuda(), idx)
    got = host(idx)
    rank = np.lexsort((np.arange(nv), -np.where(number, sv, -np.inf)))  # numbers by value, then the others by position
    text = np.concatenate([np.arange(ns), np.arange(ns + nv, n)])
    for l, b in enumerate(bud):
        want = np.sort(np.concatenate([text, ns + rank[:b - 8]]))
        assert np.array_equal(got[offsets[l]:offsets[l + 1]], want), (l, int(b))
    assert (got[offsets[-1]:] == -1).all()


def decode_steps(bud, heads_q, heads_kv, head_dim, reserve, steps, fill, order=None):
    """Decode steps on one workspace with given first contents, each against 64 bits.

    Outputs are means of values near 1 under probabilities of 16 bits or more: within 1e-4 of 64 bits."""
    import torch
    segments = len(bud)
    g = torch.Generator(device="cuda")
    g.manual_seed(segments)
    p = bd.make_problem(1, segments, heads_q, heads_kv, head_dim, 4, max(300, int(bud.max())), 8)
    seg = np.concatenate([[0], np.cumsum(bud.astype(np.int64) + reserve)])
    cache = [torch.randn(int(seg[-1]) * heads_kv * head_dim, generator=g, device="cuda", dtype=torch.bfloat16)
             for _ in range(2)]
    need = bd.workspace_size(p, None, bd.CALL_DECODE)
    assert (need > 0) == (segments * heads_kv <= 512)
    out = torch.empty(1, segments, heads_q, head_dim, device="cuda")
    ws = torch.randint(0, 256, (max(need, 1),), generator=g, device="cuda", dtype=torch.uint8)
    if fill == "ones":
        ws.fill_(255)
    for step in range(steps):
        q, kn, vn = (torch.randn(1, segments, h, head_dim, generator=g, device="cuda", dtype=torch.bfloat16)
                     for h in (heads_q, heads_kv, heads_kv))
        out.fill_(float("nan"))
        bd.tgvkv_decode_attn(p, None, *cache, torch.from_numpy(bud).cuda(), torch.from_numpy(seg).cuda(), reserve,
                             step, q, kn, vn, out, ws,
                             unit_order=None if order is None else torch.from_numpy(order).cuda())
        for l in range(segments):
            n, cap = int(bud[l]) + step + 1, int(bud[l]) + reserve
            k, v = (c[seg[l] * heads_kv * head_dim:seg[l + 1] * heads_kv * head_dim].view(heads_kv, cap, head_dim)
                    [:, :n].double() for c in cache)
            assert torch.equal(k[:, -1], kn[0, l].double())
            z = torch.matmul(q[0, l].double().view(heads_kv, -1, head_dim), k.transpose(1, 2).contiguous())
            want = torch.matmul(torch.softmax(z / head_dim ** 0.5, -1), v).view(heads_q, head_dim)
            assert (out[0, l].double() - want).abs().max().item() <= 1e-4, (fill, step, l)


@pytest.mark.parametrize("heads_q,heads_kv,head_dim", [(2, 2, 128), (4, 2, 64), (8, 2, 128), (14, 2, 128), (16, 1, 64)])
@pytest.mark.parametrize("segments", [1, 9, 16, 43, 64, 65, 128, 129, 170, 171, 256, 257])
def test_split_decode(lib, segments, heads_q, heads_kv, head_dim):
    """Decode around the unit counts where the workgroups per unit change (up to 512 units have more than one), the
    partials combined by the unit's last workgroup: any first contents of the workspace, and call after call on it."""
    log(f"split decode {segments} segments {heads_q}/{heads_kv} d{head_dim}")
    bud = np.random.default_rng(segments).integers(0, 200, segments).astype(np.int32)
    bud[0] = 0
    for fill in ("random", "ones"):
        decode_steps(bud, heads_q, heads_kv, head_dim, 3, 3, fill)


@pytest.mark.parametrize("heads_q,heads_kv,head_dim", [(4, 4, 128), (28, 4, 128), (8, 4, 64)])
@pytest.mark.parametrize("segments,rows", [(33, 1500), (42, 2000), (100, 1100), (128, 1300)])
def test_decode_units_of_even_lengths_stay_whole(lib, segments, rows, heads_q, heads_kv, head_dim):
    """129 to 512 units of equal lengths are not split (that costs up to a fifth): the same bits as in a call of more
    than 512 units, which has no splits; one unit of eight times the length and more, and they are."""
    import torch
    log(f"even decode {segments} segments of {rows} rows {heads_q}/{heads_kv} d{head_dim}")
    g = torch.Generator(device="cuda")
    g.manual_seed(segments)
    many, reserve, last = 130, 2, 9000
    p = lambda n: bd.make_problem(1, n, heads_q, heads_kv, head_dim, 4, last, 8)
    total = heads_kv * head_dim * (many * (rows + reserve) + last)
    cache = [torch.randn(total, generator=g, device="cuda", dtype=torch.bfloat16) for _ in range(2)]
    q, kn, vn = (torch.randn(1, many, h, head_dim, generator=g, device="cuda", dtype=torch.bfloat16)
                 for h in (heads_q, heads_kv, heads_kv))

    def decode(n, longest=0):
        bud = np.full(n, rows, np.int32)
        if longest:
            bud[-1] = longest
        seg = np.concatenate([[0], np.cumsum(bud.astype(np.int64) + reserve)])
        out = torch.full((1, n, heads_q, head_dim), float("nan"), device="cuda")
        ws = torch.zeros(max(bd.workspace_size(p(n), None, bd.CALL_DECODE), 1), device="cuda", dtype=torch.uint8)
        part = [t[:, :n].contiguous() for t in (q, kn, vn)]
        bd.tgvkv_decode_attn(p(n), None, *cache, torch.from_numpy(bud).cuda(), torch.from_numpy(seg).cuda(), reserve,
                             0, *part, out, ws)
        return out

    whole = decode(many)
    assert torch.equal(decode(segments), whole[:, :segments])
    split = decode(segments, last)[:, :segments - 1]
    assert (split - whole[:, :segments - 1]).abs().max().item() <= 2e-4  # each within 1e-4 of 64 bits
    assert not torch.equal(split, whole[:, :segments - 1])


@pytest.mark.parametrize("heads_q,heads_kv,layers", [(2, 1, 11), (8, 1, 11), (8, 4, 3)])
def test_idle_sequences_do_not_split_the_others(lib, heads_q, heads_kv, layers):
    """Paged decode, each sequence at its own step: a long one that does not decode leaves the others whole, the same
    bits as without it; decoding, it has them split, each output within 1e-4 of 64 bits."""
    import torch
    log(f"idle long sequence {heads_q}/{heads_kv} {layers} layers")
    g = torch.Generator(device="cuda")
    g.manual_seed(layers)
    batch, rows, last, reserve, page, D = 24 if heads_kv == 1 else 12, 1100, 8000, 4, 64, 128
    n = batch * layers
    width = -(-(last + reserve) // page)
    p = bd.make_problem(batch, layers, heads_q, heads_kv, D, 1, 0, 0)
    short = -(-(rows + reserve) // page)  # pages of a short segment; the last sequence's have `width` each
    pages = (n - layers) * short + layers * width
    table = np.full((n, width), -1, np.int32)
    ids = np.random.default_rng(layers).permutation(pages).astype(np.int32)
    for s in range(n):
        first = min(s, n - layers) * short + max(s - (n - layers), 0) * width
        table[s, :short if s < n - layers else width] = ids[first:first + (short if s < n - layers else width)]
    k, v = (torch.randn(pages, heads_kv, page, D, generator=g, device="cuda", dtype=torch.bfloat16) for _ in range(2))
    q, kn, vn = (torch.randn(batch, layers, h, D, generator=g, device="cuda", dtype=torch.bfloat16)
                 for h in (heads_q, heads_kv, heads_kv))
    steps = np.arange(batch, dtype=np.int32) % reserve

    def decode(longest, idle):
        bud = np.full(n, rows, np.int32)
        bud[n - layers:] = longest
        st = steps.copy()
        if idle:
            st[-1] = -1
        out = torch.full((batch, layers, heads_q, D), float("nan"), device="cuda")
        ws = torch.zeros(max(bd.workspace_size(p, None, bd.CALL_DECODE), 1), device="cuda", dtype=torch.uint8)
        kc, vc = k.clone(), v.clone()
        bd.tgvkv_decode_attn_paged(p, None, kc, vc, page, torch.from_numpy(table).cuda(), torch.from_numpy(bud).cuda(),
                                   reserve, torch.from_numpy(st).cuda(), q, kn, vn, out, ws)
        for b in range(batch - 1 if idle else batch):
            for l in range(layers):
                m = int(bud[b * layers + l]) + int(st[b]) + 1
                at = torch.from_numpy(table[b * layers + l, :-(-m // page)].astype(np.int64)).cuda()
                K, V = (c[at].transpose(0, 1).reshape(heads_kv, -1, D)[:, :m].double() for c in (kc, vc))
                assert torch.equal(K[:, -1], kn[b, l].double())
                z = torch.matmul(q[b, l].double().view(heads_kv, -1, D), K.transpose(1, 2).contiguous())
                want = torch.matmul(torch.softmax(z / D ** 0.5, -1), V).view(heads_q, D)
                assert (out[b, l].double() - want).abs().max().item() <= 1e-4, (longest, idle, b, l)
        return out[:-1]

    even = decode(rows, False)
    assert torch.equal(decode(last, True), even)
    assert not torch.equal(decode(last, False), even)


@pytest.mark.parametrize("heads_q,heads_kv,head_dim", [(4, 4, 128), (4, 2, 64), (28, 4, 128), (32, 4, 64)])
@pytest.mark.parametrize("segments", [5, 33, 56, 75, 128])
def test_split_decode_of_uneven_lengths(lib, segments, heads_q, heads_kv, head_dim):
    """Units of one row to several thousand in one call, longest first as a budget call orders them and in no order:
    each takes its own number of splits, the lengths where it changes among them."""
    log(f"uneven split decode {segments} segments {heads_q}/{heads_kv} d{head_dim}")
    r = np.random.default_rng(segments)
    bud = np.exp(r.uniform(0, np.log(5000), segments)).astype(np.int32)
    edges = [0, 1021, 1023, 1024, 2047, 2048, 5000]  # rows of a call: budget + step + 1
    bud[r.permutation(segments)[:len(edges)]] = edges[:segments]
    for order in (np.argsort(-bud, kind="stable").astype(np.int32), None):
        decode_steps(bud, heads_q, heads_kv, head_dim, 2, 2, "random", order)
