"""Calls of more sequences than one batch holds: the last group of them is smaller, with the splits of the whole one.  Its steps
give the bits of separate launches whatever form they take."""
import pytest

pytestmark = pytest.mark.gpu

from paper_2511_20100_amd import inputs

V = 1040
SHAPES = {
    "1p5b": inputs.POLICY_1P5B.with_(n_layers=2, vocab=V),
    "7b": inputs.POLICY_7B.with_(n_layers=1, vocab=V),
    "mha": inputs.POLICY_1P3B_MHA.with_(n_layers=1, vocab=V),
    # the splits of 128 rows are a round of workgroups here, too
    "narrow": inputs.ModelConfig(2, 1536, 12, 2, 128, 512, V, dtype="bf16"),
}


@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("n_prompts,n_samples", [(129, 1), (144, 1), (160, 1), (34, 5), (24, 8)])  # the last: 1, 16, 32, 45, 64 rows
def test_the_last_group(shape, n_prompts, n_samples):
    import numpy as np
    import torch
    from paper_2511_20100_amd import mtmc as lib
    cfg = SHAPES[shape]
    handle = lib.mtmc_weights_create(lib.make_config(cfg, 128), inputs.make_weights(cfg, seed=0, std=0.04, gain_std=0.1).blob())
    try:
        prompts = torch.from_numpy(inputs.make_prompts(n_prompts, 20, cfg.vocab, seed=3)).cuda()
        lens = torch.from_numpy(np.random.default_rng(1).integers(1, 21, n_prompts).astype(np.int32)).cuda()
        got = []
        for limit in (0, 10_000_000):
            lib.mtmc_set_option(handle, lib.MTMC_OPT_PERSISTENT_DECODE, limit)
            got.append([t.cpu() for t in lib.mtmc_rollout(handle, prompts, n_samples, 5, 1.0, 3)] +
                       [t.cpu() for t in lib.mtmc_rollout_ragged(handle, prompts, lens, n_samples, 5, 1.0, 3)])
            lib.mtmc_poll_errors(handle)
        assert all(torch.equal(a, b) for a, b in zip(*got))
    finally:
        lib.mtmc_weights_destroy(handle)
