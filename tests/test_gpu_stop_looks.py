"""Looks at the stop flags where the caller has not said how often: the results of looks every that many steps, and of calls that
follow each other without a wait."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

from paper_2511_20100_amd import inputs

V = 64


def test_the_choice_can_be_given_back():
    """A call of 65 tokens: not packed unless a period is set, which changes bits; the library's choice, set again, is the one it
    began with, and so are the bits.  Other values below zero are refused as ever."""
    import torch
    from paper_2511_20100_amd import mtmc as lib
    cfg = inputs.ModelConfig(2, 256, 4, 2, 128, 688, V, dtype="bf16")
    handle = lib.mtmc_weights_create(lib.make_config(cfg, 256), inputs.make_weights(cfg, seed=0, std=0.05, gain_std=0.1).blob())
    try:
        lens = torch.from_numpy((3 + np.arange(10) * 11 % 50).astype(np.int32)).cuda()
        prompts = torch.from_numpy(inputs.make_prompts(10, 53, V, seed=2)).cuda()
        got = []
        for value in (None, 2, lib.MTMC_STOP_POLL_CHOOSE):
            if value is not None:
                lib.mtmc_set_option(handle, lib.MTMC_OPT_STOP_POLL_STEPS, value)
            got.append([t.cpu() for t in lib.mtmc_rollout_ragged(handle, prompts, lens, 5, 65, 1.0, 1, stop_id=3)])
            lib.mtmc_poll_errors(handle)
        assert all(torch.equal(a, b) for a, b in zip(got[0], got[2]))
        assert not torch.equal(got[0][1], got[1][1])
        for value in (-2, -(1 << 31), (1 << 20) + 1):
            with pytest.raises(lib.MtmcError, match="STOP_POLL"):
                lib.mtmc_set_option(handle, lib.MTMC_OPT_STOP_POLL_STEPS, value)
    finally:
        lib.mtmc_weights_destroy(handle)


@pytest.mark.parametrize("layers,steps", [(2, 8), (6, 4)])
def test_steps_that_the_library_chooses(layers, steps):
    import torch
    from paper_2511_20100_amd import mtmc as lib
    cfg = inputs.ModelConfig(layers, 256, 4, 2, 128, 688, V, dtype="bf16")
    blob = inputs.make_weights(cfg, seed=0, std=0.05, gain_std=0.1).blob()
    lens = torch.from_numpy((3 + np.arange(10) * 11 % 50).astype(np.int32)).cuda()
    prompts = torch.from_numpy(inputs.make_prompts(10, 53, V, seed=2)).cuda()
    got = []
    for value in (None, steps):
        handle = lib.mtmc_weights_create(lib.make_config(cfg, 256), blob)
        if value:
            lib.mtmc_set_option(handle, lib.MTMC_OPT_STOP_POLL_STEPS, value)
        got.append([t.cpu() for t in lib.mtmc_rollout_ragged(handle, prompts, lens, 5, 70, 1.0, 1, stop_id=3)])
        lib.mtmc_poll_errors(handle)
        lib.mtmc_weights_destroy(handle)
    assert all(torch.equal(a, b) for a, b in zip(*got))
    ends = np.sort(got[0][2].numpy())
    assert ends[17] < 40 and ends[-1] > 4 * steps  # tiles were freed while rows still ran


def test_calls_in_turn_on_two_streams():
    """Nobody waits for a call but the looks of the next one, which are on the other stream, at the same place of the host's memory."""
    import torch
    from paper_2511_20100_amd import mtmc as lib
    cfg = inputs.ModelConfig(6, 256, 4, 2, 128, 688, V, dtype="bf16")
    handle = lib.mtmc_weights_create(lib.make_config(cfg, 256), inputs.make_weights(cfg, seed=0, std=0.05, gain_std=0.1).blob())
    try:
        lens = torch.full((4,), 20, dtype=torch.int32, device="cuda")
        prompts = torch.from_numpy(inputs.make_prompts(4, 20, V, seed=2)).cuda()
        size = lib.mtmc_rollout_ragged_workspace_bytes(handle, 4, 20, 4, 100)
        spaces = [torch.empty(size, dtype=torch.uint8, device="cuda") for _ in range(2)]
        streams = [torch.cuda.Stream() for _ in range(2)]

        def run(i, seed):
            with torch.cuda.stream(streams[i]):
                return lib.mtmc_rollout_ragged(handle, prompts, lens, 4, 100, 1.0, seed, stop_id=3, workspace=spaces[i],
                                               stream=streams[i])

        torch.cuda.synchronize()
        want = []
        for seed in range(3):
            outs = run(0, seed)
            torch.cuda.synchronize()
            want.append([t.cpu() for t in outs])
        got = [(i % 3, run(i % 2, i % 3)) for i in range(70)]
        torch.cuda.synchronize()
        lib.mtmc_poll_errors(handle)
        for i, (seed, outs) in enumerate(got):
            assert all(torch.equal(a, b.cpu()) for a, b in zip(want[seed], outs)), i
    finally:
        lib.mtmc_weights_destroy(handle)


def test_a_short_call_only_enqueues():
    """Up to 65 tokens, a stop token among them: the call returns while the stream still has other work ahead of it."""
    import torch
    from paper_2511_20100_amd import mtmc as lib
    cfg = inputs.ModelConfig(6, 256, 4, 2, 128, 688, V, dtype="bf16")
    handle = lib.mtmc_weights_create(lib.make_config(cfg, 256), inputs.make_weights(cfg, seed=0, std=0.05, gain_std=0.1).blob())
    try:
        lens = torch.full((4,), 20, dtype=torch.int32, device="cuda")
        prompts = torch.from_numpy(inputs.make_prompts(4, 20, V, seed=2)).cuda()
        for new in (40, 64, 65):
            ws = torch.empty(lib.mtmc_rollout_ragged_workspace_bytes(handle, 4, 20, 4, new), dtype=torch.uint8, device="cuda")
            want = [t.cpu() for t in lib.mtmc_rollout_ragged(handle, prompts, lens, 4, new, 1.0, 1, stop_id=3, workspace=ws)]
            a = torch.randn(16384, 16384, dtype=torch.float16, device="cuda")
            c = torch.empty_like(a)
            torch.matmul(a, a, out=c)
            torch.cuda.synchronize()
            done = torch.cuda.Event()
            for _ in range(40):  # about 0.3 s; the call is a few milliseconds of host work
                torch.matmul(a, a, out=c)
            done.record()
            got = lib.mtmc_rollout_ragged(handle, prompts, lens, 4, new, 1.0, 1, stop_id=3, workspace=ws)
            assert not done.query(), new
            torch.cuda.synchronize()
            lib.mtmc_poll_errors(handle)
            assert all(torch.equal(x, y.cpu()) for x, y in zip(want, got)), new
    finally:
        lib.mtmc_weights_destroy(handle)
