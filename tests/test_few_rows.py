"""Decode steps of few rows: those whose readers ask for all of their data (up to ASK_ROWS) and those above the line, one block and
more than the memory that the blocks hand on has pieces, one to eight context chunks (chunks beyond the context among them), sequences of
different lengths, some of which end."""
import os
import re

import numpy as np
import pytest

from paper_2511_20100_amd import inputs
from test_persistent_turn import CSRC, _run

V = 1040
with open(os.path.join(CSRC, "persistent_cut.h")) as f:
    ASK_ROWS = int(re.search(r"kPersistAskRows = (\d+);", f.read()).group(1))
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


def _same_bits(shape, calls):
    """Prompts of one length and of different ones, of which some sequences end: separate launches against one."""
    import torch
    from paper_2511_20100_amd import mtmc as lib
    cfg = SHAPES[shape]
    handle = lib.mtmc_weights_create(lib.make_config(cfg, 2400), inputs.make_weights(cfg, seed=0, std=0.04, gain_std=0.1).blob())
    try:
        for n_prompts, plen, n_samples, max_new in calls:
            prompts = torch.from_numpy(inputs.make_prompts(n_prompts, plen, cfg.vocab, seed=plen)).cuda()
            drawn = np.random.default_rng(plen).integers(1, plen + 1, n_prompts).astype(np.int32)
            for lens in (drawn, np.minimum(drawn, max(1, plen // 3))):  # the second: chunks beyond every context
                lens = torch.from_numpy(lens).cuda()
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


@pytest.mark.gpu
@pytest.mark.parametrize("shape", SHAPES)
def test_rows_on_both_sides_of_the_line(shape):
    _same_bits(shape, ((1, 3, 3, 40), (3, 250, 1, 20), (1, 1500, 4, 9), (2, 2000, 2, 6), (5, 40, 1, 9), (1, 5, 2, 200), (3, 200, 4, 9),
                       (1, 40, ASK_ROWS, 9), (1, 40, ASK_ROWS + 1, 9)))


@pytest.mark.gpu
@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("rows", range(1, ASK_ROWS + 1))
def test_rows_that_ask_for_everything(shape, rows):
    """1, 3, 5 and 8 chunks with two kv heads, sequences of one prompt and of a prompt each."""
    calls = [(1, plen, rows, max_new) for plen, max_new in ((3, 40), (250, 20), (600, 8), (2000, 6))]
    _same_bits(shape, calls + ([(rows, 300, 1, 12), (rows, 1100, 1, 6)] if rows > 1 else []))
