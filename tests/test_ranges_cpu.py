"""The bound of test_gpu_ranges.py tells a wrong share from a right one (host only, on the oracle)."""

import numpy as np
import pytest

import oracle.tgvkv_oracle as O
from tests.test_gpu_ranges import SCORE_BOUND, SPLIT_STATS
from workloads import bf16_bits_to_f32, make_prefill_tensors
from workloads.configs import custom_config


@pytest.mark.parametrize("name", sorted(SPLIT_STATS))
def test_every_key_shows_in_the_normalisers(name):
    """Left out or counted twice, each single key of test_split_statistics moves the normaliser of some
    row of one query head by twice the bound."""
    cfg = custom_config(name=name, **dict(dict(batch=1, layers=2), **SPLIT_STATS[name]))
    t = make_prefill_tensors(cfg, seed=5, names=("q_text", "k"))
    for l in range(cfg.layers):
        k = bf16_bits_to_f32(t["k"][0, l])
        for h in range(0, cfg.heads_q, cfg.heads_q // cfg.heads_kv):
            g = h * cfg.heads_kv // cfg.heads_q
            P, _ = O.text_row_softmax(bf16_bits_to_f32(t["q_text"][0, l, h:h + 1]), k[g:g + 1], cfg.n_sys, cfg.n_vis,
                                      cfg.n_qst, O.default_scale(cfg.head_dim))
            rows = P[0, cfg.n_sys:]  # the question rows, whose sums the sweep takes
            most = np.minimum(-np.log1p(-np.minimum(rows, 0.99)), np.log1p(rows)).max(0)
            assert most.min() > 2 * SCORE_BOUND, (l, g, int(most.argmin()), most.min())
