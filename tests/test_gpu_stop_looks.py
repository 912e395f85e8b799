"""Looks at the stop flags where the caller has not said how often: the results of looks every that many steps, and looks of a call
that has ended do not reach the next one."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

from paper_2511_20100_amd import inputs

V = 64


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


def test_calls_one_after_the_other_on_two_streams():
    """The first call's last look (nobody runs any more) is written after the call has returned."""
    import torch
    from paper_2511_20100_amd import mtmc as lib
    cfg = inputs.ModelConfig(6, 256, 4, 2, 128, 688, V, dtype="bf16")
    handle = lib.mtmc_weights_create(lib.make_config(cfg, 256), inputs.make_weights(cfg, seed=0, std=0.05, gain_std=0.1).blob())
    try:
        lens = torch.full((4,), 20, dtype=torch.int32, device="cuda")
        prompts = torch.from_numpy(inputs.make_prompts(4, 20, V, seed=2)).cuda()
        run = lambda ws, st, **kw: lib.mtmc_rollout_ragged(handle, prompts, lens, 4, 100, 1.0, 1, stop_id=3, workspace=ws, **kw)
        size = lib.mtmc_rollout_ragged_workspace_bytes(handle, 4, 20, 4, 100)
        spaces = [torch.empty(size, dtype=torch.uint8, device="cuda") for _ in range(2)]
        streams = [torch.cuda.Stream() for _ in range(2)]
        want = [t.cpu() for t in run(spaces[0], None)]
        torch.cuda.synchronize()
        for i in range(8):
            with torch.cuda.stream(streams[i % 2]):
                got = run(spaces[i % 2], None, stream=streams[i % 2])
            streams[i % 2].synchronize()
            assert all(torch.equal(a, b.cpu()) for a, b in zip(want, got)), i
    finally:
        lib.mtmc_weights_destroy(handle)
