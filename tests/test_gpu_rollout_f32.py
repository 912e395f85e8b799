"""fp32 generation as one launch: the bits of the launches of its own, for one row and several blocks of eight, small and large vocabularies,
both head sizes, contexts over several rounds of keys, stop tokens, and with a wait that gives up."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

from paper_2511_20100_amd import inputs

SHAPES = {
    "tiny": (inputs.TINY, [(1, 1, 1, 2), (4, 32, 2, 33), (3, 250, 3, 20), (4, 17, 4, 9), (5, 17, 5, 4)]),   # 1, 8, 9, 16, 25 rows
    "small": (inputs.ModelConfig(1, 32, 4, 1, 64, 48, 48, dtype="fp32"), [(1, 3, 1, 40), (2, 300, 4, 12), (1, 390, 2, 5)]),
    "hd128": (inputs.ModelConfig(3, 272, 2, 2, 128, 2032, 1040, dtype="fp32"), [(2, 20, 3, 10), (5, 6, 4, 5)]),
    "wide": (inputs.ModelConfig(2, 1280, 20, 5, 64, 1296, 8000, dtype="fp32"), [(1, 40, 1, 6), (2, 5, 8, 4)]),
    # does not fit: five queries per kv head; an operand of 2048 values; a vocabulary that takes the tiles
    "separate": (inputs.ModelConfig(1, 64, 5, 1, 64, 64, 112, dtype="fp32"), [(2, 9, 2, 6)]),
    "separate-wide": (inputs.ModelConfig(1, 64, 1, 1, 64, 2048, 112, dtype="fp32"), [(2, 9, 2, 6)]),
    "separate-vocab": (inputs.ModelConfig(1, 64, 1, 1, 64, 64, 9008, dtype="fp32"), [(2, 9, 2, 6)]),
}


@pytest.fixture(scope="module")
def lib():
    from paper_2511_20100_amd import mtmc
    return mtmc


@pytest.fixture(scope="module", params=SHAPES)
def policy(request, lib):
    cfg, calls = SHAPES[request.param]
    handle = lib.mtmc_weights_create(lib.make_config(cfg, 512), inputs.make_weights(cfg, seed=0, std=0.06, gain_std=0.1).blob())
    yield cfg, calls, handle, not request.param.startswith("separate")
    lib.mtmc_weights_destroy(handle)


def test_the_bits_of_separate_launches(lib, policy):
    import torch
    cfg, calls, handle, fits = policy
    for n_prompts, plen, n_samples, max_new in calls:
        prompts = torch.from_numpy(inputs.make_prompts(n_prompts, plen, cfg.vocab, seed=plen)).cuda()
        got = []
        for value in (0, 10_000_000):
            lib.mtmc_set_option(handle, lib.MTMC_OPT_PERSISTENT_DECODE, value)
            for temperature in (1.0, 0.0):
                got.append([t.cpu() for t in lib.mtmc_rollout(handle, prompts, n_samples, max_new, temperature, 3)])
                lib.mtmc_poll_errors(handle)
        for a, b in zip(got[:2], got[2:]):
            assert all(torch.equal(x, y) for x, y in zip(a, b)), (n_prompts, plen, n_samples, max_new)
        assert torch.isfinite(got[0][1]).all()


def test_stop_tokens_and_lengths(lib, policy):
    import torch
    cfg, _, handle, _ = policy
    lens = torch.from_numpy(np.random.default_rng(2).integers(1, 50, 5).astype(np.int32)).cuda()
    prompts = torch.from_numpy(inputs.make_prompts(5, 50, cfg.vocab, seed=5)).cuda()
    free = lib.mtmc_rollout_ragged(handle, prompts, lens, 2, 12, 1.0, 4)[0].cpu().numpy()
    stop = int(free[0, 4])
    outs = []
    for value in (0, 10_000_000):
        lib.mtmc_set_option(handle, lib.MTMC_OPT_PERSISTENT_DECODE, value)
        outs.append([t.cpu() for t in lib.mtmc_rollout_ragged(handle, prompts, lens, 2, 12, 1.0, 4, stop_id=stop)])
        lib.mtmc_poll_errors(handle)
    assert all(torch.equal(a, b) for a, b in zip(*outs))
    assert int(outs[0][2][0]) <= 5


def test_a_wait_that_gives_up(lib, policy):
    """... is reported, and nothing of it is left; this also shows which shapes the one launch takes."""
    import torch
    cfg, _, handle, fits = policy
    prompts = torch.from_numpy(inputs.make_prompts(2, 9, cfg.vocab, seed=1)).cuda()
    ref = [t.cpu() for t in lib.mtmc_rollout(handle, prompts, 2, 6, 1.0, 3)]
    lib.mtmc_set_option(handle, lib.MTMC_OPT_PERSISTENT_DECODE, 1)
    try:
        lib.mtmc_rollout(handle, prompts, 2, 6, 1.0, 3)
        if fits:
            with pytest.raises(lib.MtmcError, match="persistent"):
                lib.mtmc_poll_errors(handle)
        else:
            lib.mtmc_poll_errors(handle)
    finally:
        lib.mtmc_set_option(handle, lib.MTMC_OPT_PERSISTENT_DECODE, 10_000_000)
    again = [t.cpu() for t in lib.mtmc_rollout(handle, prompts, 2, 6, 1.0, 3)]
    lib.mtmc_poll_errors(handle)
    assert all(torch.equal(a, b) for a, b in zip(ref, again))
