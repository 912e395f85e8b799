"""More shapes than the cache of decode-step graphs holds: calls give what they give without graphs, from two threads as
from one, and a graph that makes room is not waited for with the whole device."""
import threading

import pytest

pytestmark = pytest.mark.gpu

from paper_2511_20100_amd import inputs

SMALL = inputs.ModelConfig(2, 256, 4, 2, 64, 512, 1040, dtype="bf16")
PLENS = [9, 14, 20, 33, 40, 47]
NEW = 12


@pytest.fixture(scope="module")
def lib():
    from paper_2511_20100_amd import mtmc
    return mtmc


def _handle(lib, cfg):
    return lib.mtmc_weights_create(lib.make_config(cfg, 128), inputs.make_weights(cfg, seed=0, std=0.05, gain_std=0.1).blob())


@pytest.mark.parametrize("cfg", [inputs.TINY, SMALL], ids=["fp32", "bf16"])
def test_two_threads_with_six_shapes_each(lib, cfg):
    import torch
    handle = _handle(lib, cfg)
    try:
        shapes = [(n, plen) for n in (2, 3) for plen in PLENS]  # a thread's shapes: one n
        prompts = {s: torch.from_numpy(inputs.make_prompts(*s, cfg.vocab, seed=sum(s))).cuda() for s in shapes}
        wss = {s: torch.empty(lib.mtmc_rollout_workspace_bytes(handle, *s, 2, NEW), dtype=torch.uint8, device="cuda") for s in shapes}
        streams = {n: torch.cuda.Stream() for n in (2, 3)}

        def call(s, seed, stream=None):
            return lib.mtmc_rollout(handle, prompts[s], 2, NEW, 1.0, seed, workspace=wss[s], stream=stream)

        lib.mtmc_set_option(handle, lib.MTMC_OPT_HIP_GRAPH, 0)
        ref = {(s, seed): [t.cpu() for t in call(s, seed)] for s in shapes for seed in range(4)}
        lib.mtmc_set_option(handle, lib.MTMC_OPT_HIP_GRAPH, 1)
        torch.cuda.synchronize()
        got, failed = {}, []

        def work(n):
            try:
                with torch.cuda.stream(streams[n]):
                    for seed in range(4):
                        for s in shapes:
                            if s[0] == n:
                                got[s, seed] = call(s, seed, streams[n])
            except Exception as e:  # noqa: BLE001  (reported by the test's own thread)
                failed.append(e)

        threads = [threading.Thread(target=work, args=(n,)) for n in (2, 3)]
        for t in threads:
            t.start()
        for t in threads:
            t.join()
        torch.cuda.synchronize()
        lib.mtmc_poll_errors(handle)
        assert not failed, failed
        assert got.keys() == ref.keys()
        for k, pair in ref.items():
            assert all(torch.equal(a, b.cpu()) for a, b in zip(pair, got[k])), k
    finally:
        lib.mtmc_weights_destroy(handle)


def test_a_new_shape_does_not_wait_for_other_streams(lib):
    import torch
    handle = _handle(lib, inputs.TINY)
    try:
        shapes = [(n, plen) for n in (1, 2) for plen in PLENS]
        prompts = {s: torch.from_numpy(inputs.make_prompts(*s, inputs.TINY.vocab, seed=1)).cuda() for s in shapes}
        wss = {s: torch.empty(lib.mtmc_rollout_workspace_bytes(handle, *s, 1, NEW), dtype=torch.uint8, device="cuda") for s in shapes}
        a = torch.randn(16384, 16384, dtype=torch.float16, device="cuda")
        c = torch.empty_like(a)
        torch.matmul(a, a, out=c)
        torch.cuda.synchronize()
        other, done = torch.cuda.Stream(), torch.cuda.Event()
        with torch.cuda.stream(other):
            for _ in range(200):  # about 1.5 s; the calls below are a few milliseconds of host work each
                torch.matmul(a, a, out=c)
            done.record()
        for s in shapes:
            lib.mtmc_rollout(handle, prompts[s], 1, NEW, 1.0, 1, workspace=wss[s])
        assert not done.query()
        torch.cuda.synchronize()
        lib.mtmc_poll_errors(handle)
    finally:
        lib.mtmc_weights_destroy(handle)
