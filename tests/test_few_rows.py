"""Decode steps of few rows, whose readers ask for the data: the rows on both sides of the line to the counters, one block and
several, one to eight context chunks (a chunk beyond the context among them), sequences of different lengths, some of which end."""
import numpy as np
import pytest

from paper_2511_20100_amd import inputs
from test_persistent_turn import _run

V = 1040
SHAPES = {
    "one-block": inputs.POLICY_1P5B.with_(n_layers=1, vocab=V),
    "1p5b": inputs.POLICY_1P5B.with_(n_layers=7, vocab=V),  # more blocks than pieces of memory that they hand on
    "7b": inputs.POLICY_7B.with_(n_layers=2, vocab=V),
    # workgroups that have nothing but a unit of the attention
    "narrow": inputs.ModelConfig(6, 1536, 12, 2, 128, 512, V, dtype="bf16"),
    "one-kv-head": inputs.ModelConfig(2, 1568, 8, 1, 128, 1104, V, dtype="bf16"),  # eight chunks; padded widths
}


def test_the_buffers_of_a_block_lie_apart(tmp_path):
    _run(tmp_path, "persistent_hand_check")


def test_nobody_finds_an_earlier_or_a_later_block_in_a_place(tmp_path):
    _run(tmp_path, "persistent_order_check")


@pytest.mark.gpu
@pytest.mark.parametrize("shape", SHAPES)
def test_rows_on_both_sides_of_the_line(shape):
    import torch
    from paper_2511_20100_amd import mtmc as lib
    cfg = SHAPES[shape]
    handle = lib.mtmc_weights_create(lib.make_config(cfg, 2400), inputs.make_weights(cfg, seed=0, std=0.04, gain_std=0.1).blob())
    try:
        for n_prompts, plen, n_samples, max_new in ((1, 3, 3, 40), (3, 250, 1, 20), (1, 1500, 4, 9), (2, 2000, 2, 6), (5, 40, 1, 9), (1, 5, 2, 200), (3, 200, 4, 9)):
            prompts = torch.from_numpy(inputs.make_prompts(n_prompts, plen, cfg.vocab, seed=plen)).cuda()
            lens = torch.from_numpy(np.random.default_rng(plen).integers(1, plen + 1, n_prompts).astype(np.int32)).cuda()
            got, stop = [], -1
            for value in (0, 10_000_000):
                lib.mtmc_set_option(handle, lib.MTMC_OPT_PERSISTENT_DECODE, value)
                outs = list(lib.mtmc_rollout(handle, prompts, n_samples, max_new, 1.0, 3))
                if stop < 0:  # a token that the second step of some sequence gives
                    stop = int(outs[0][0, 1])
                outs += lib.mtmc_rollout_ragged(handle, prompts, lens, n_samples, max_new, 1.0, 4, stop_id=stop)
                got.append([t.cpu() for t in outs])
                lib.mtmc_poll_errors(handle)
            assert all(torch.equal(a, b) for a, b in zip(*got)), (n_prompts, plen, n_samples, max_new)
    finally:
        lib.mtmc_weights_destroy(handle)
