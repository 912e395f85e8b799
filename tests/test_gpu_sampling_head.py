"""The persistent sampling LM head of 65 to 128 rows: the fewest and the most rows, entries that leave the last block of
128 partly empty, the shortest reduction that it takes, and the form that it replaces just below its range.  Every chosen
row is replayed on the oracle."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

from parity import LOGP_TOL_BF16, check_ragged_by_replay, check_rollout_by_replay
from paper_2511_20100_amd import inputs


@pytest.fixture(scope="module")
def lib():
    from paper_2511_20100_amd import mtmc
    return mtmc


# 32768 entries: one block of 128 per CU; 32752: below it; 65584 = 512 blocks and three tiles of 16: two blocks for some
@pytest.mark.parametrize("d,heads,vocab,n_prompts,n_samples", [(256, 2, 32768, 13, 5), (256, 2, 65584, 16, 8),
                                                                (128, 1, 40016, 9, 9), (256, 2, 32752, 16, 8)])
def test_rows_and_vocabulary_edges(lib, d, heads, vocab, n_prompts, n_samples):
    import torch
    cfg = inputs.ModelConfig(1, d, heads, 1, 128, 512, vocab, dtype="bf16")
    w = inputs.make_weights(cfg, seed=0, std=0.05, gain_std=0.1)
    handle = lib.mtmc_weights_create(lib.make_config(cfg, 128), w.blob())
    try:
        prompts = inputs.make_prompts(n_prompts, 18, cfg.vocab, seed=2)
        last = n_prompts * n_samples - 1
        rep = check_rollout_by_replay(handle, w, prompts, n_samples, 4, 1.0, 1, max_positions=128,
                                      rows=[0, n_samples, 63, last], label=f"{vocab}")
        # the same prompts in a call of few rows (another kernel): both within the tolerance of the exact value
        alone = lib.mtmc_rollout(handle, torch.from_numpy(prompts[:2]).cuda(), n_samples, 4, 1.0, 1)
        same = (alone[0].cpu().numpy() == rep["ids"][:2 * n_samples]).all(axis=1)
        assert same.any()
        assert np.abs(alone[1].cpu().numpy() - rep["logprobs"][:2 * n_samples])[same].max() <= 2 * LOGP_TOL_BF16
        greedy = lib.mtmc_rollout(handle, torch.from_numpy(prompts).cuda(), n_samples, 3, 0.0, 1)
        rows = greedy[0].cpu().numpy().reshape(n_prompts, n_samples, 3)
        assert (rows == rows[:, :1]).all()  # the samples of a prompt agree where nothing is drawn
    finally:
        lib.mtmc_weights_destroy(handle)


def test_rows_that_end(lib):
    cfg = inputs.ModelConfig(1, 256, 2, 1, 128, 512, 33008, dtype="bf16")
    w = inputs.make_weights(cfg, seed=0, std=0.05, gain_std=0.1)
    handle = lib.mtmc_weights_create(lib.make_config(cfg, 128), w.blob())
    try:
        lens = np.arange(5, 25, dtype=np.int32)
        prompts = inputs.make_prompts(len(lens), int(lens.max()), cfg.vocab, seed=2)
        check_ragged_by_replay(handle, w, prompts, lens, 5, 6, 1.0, 1, stop_id=3, max_positions=128, label="ragged")
    finally:
        lib.mtmc_weights_destroy(handle)
