"""Persistent launches that do not get the whole device in time: the workgroups that are there do the work, with the bits of the
separate launches.  Forced by a limit of a microsecond, and by another stream's kernel that holds a part of the device for a while."""
import pytest

pytestmark = pytest.mark.gpu

from paper_2511_20100_amd import inputs

V = 1040
SHAPES = {
    "narrow": inputs.ModelConfig(3, 1536, 12, 2, 128, 512, V, dtype="bf16"),
    "1p5b": inputs.POLICY_1P5B.with_(n_layers=2, vocab=V),
    "7b": inputs.POLICY_7B.with_(n_layers=1, vocab=V),
    "mha": inputs.POLICY_1P3B_MHA.with_(n_layers=2, vocab=V),
    "wide-kv": inputs.ModelConfig(2, 1600, 16, 8, 128, 1104, V, dtype="bf16"),
    # one tile of rows, the other cuts: gate / up tiles per workgroup and ranges of the down projection
    "4x5": inputs.ModelConfig(2, 1536, 12, 2, 128, 6144, V, dtype="bf16"),
    "4x4": inputs.ModelConfig(2, 3584, 28, 4, 128, 8192, V, dtype="bf16"),
    "6x8": inputs.ModelConfig(2, 2048, 16, 2, 128, 11008, V, dtype="bf16"),
    "6x4": inputs.ModelConfig(2, 3072, 24, 8, 128, 12288, V, dtype="bf16"),
    "10x5": inputs.ModelConfig(2, 1536, 12, 2, 128, 16384, V, dtype="bf16"),
    "10x8": inputs.ModelConfig(2, 2048, 16, 2, 128, 14336, V, dtype="bf16"),
    # the widest and narrowest that take the cuts for more than one tile of rows
    "d4096": inputs.ModelConfig(1, 4096, 32, 8, 128, 20480, V, dtype="bf16"),
    "d2560": inputs.ModelConfig(2, 2560, 20, 4, 128, 18944, V, dtype="bf16"),
    "F8208": inputs.ModelConfig(2, 1536, 12, 4, 128, 8208, V, dtype="bf16"),
    "F12288": inputs.ModelConfig(2, 1536, 12, 2, 128, 12288, V, dtype="bf16"),
    # few units of the attention: up to eight context chunks with one tile of rows, seven with two, three with three
    "one-kv-head": inputs.ModelConfig(2, 1536, 8, 1, 128, 8960, V, dtype="bf16"),
    "fp32": inputs.TINY,
    "fp32-hd128": inputs.ModelConfig(3, 272, 2, 2, 128, 2032, 1040, dtype="fp32"),
}
ONE_TILE = [(1, 1, 1, 12), (1, 300, 2, 9), (2, 1100, 1, 5), (5, 90, 3, 20)]
CALLS = {
    "narrow": ONE_TILE,
    # also 18, 32, 33, 48, 49 and 64 rows, one to three context chunks
    "1p5b": ONE_TILE + [(3, 1, 6, 6), (4, 300, 8, 6), (11, 127, 3, 4), (6, 20, 8, 5), (7, 90, 7, 6), (8, 300, 8, 6), (4, 1500, 16, 3)],
    "7b": ONE_TILE + [(17, 300, 1, 6), (4, 100, 8, 5), (3, 1500, 8, 4)],
    "mha": ONE_TILE,
    "wide-kv": ONE_TILE,
    **{cut: ONE_TILE + [(2, 40, 8, 5)] for cut in ("4x5", "4x4", "6x8", "6x4", "10x5", "10x8")},
    **{shape: [(1, 300, 2, 5), (4, 100, 8, 5), (17, 20, 1, 4)] for shape in ("d4096", "d2560")},
    **{shape: [(1, 300, 2, 5), (4, 100, 8, 5), (6, 100, 8, 4), (8, 100, 8, 4), (33, 20, 1, 4)] for shape in ("F8208", "F12288")},
    "one-kv-head": [(1, 1100, 1, 4), (2, 1100, 8, 4), (17, 900, 1, 3), (5, 700, 4, 3), (33, 500, 1, 3), (6, 500, 7, 3), (8, 300, 8, 3)],
    "fp32": [(1, 1, 1, 3), (4, 32, 2, 20), (4, 17, 4, 9)],
    "fp32-hd128": [(2, 20, 3, 10)],
}


@pytest.fixture(scope="module")
def lib():
    from paper_2511_20100_amd import mtmc
    return mtmc


def _policy(lib, name):
    cfg = SHAPES[name]
    return cfg, lib.mtmc_weights_create(lib.make_config(cfg, 2400), inputs.make_weights(cfg, seed=0, std=0.04, gain_std=0.1).blob())


def _rollout(lib, handle, prompts, n_samples, max_new, limit, **kw):
    lib.mtmc_set_option(handle, lib.MTMC_OPT_PERSISTENT_DECODE, limit)
    return [t.cpu() for t in lib.mtmc_rollout(handle, prompts, n_samples, max_new, 1.0, 3, **kw)]


@pytest.mark.parametrize("shape", SHAPES)
def test_the_bits_of_separate_launches(lib, shape):
    import torch
    cfg, handle = _policy(lib, shape)
    try:
        for n_prompts, plen, n_samples, max_new in CALLS[shape]:
            prompts = torch.from_numpy(inputs.make_prompts(n_prompts, plen, cfg.vocab, seed=plen)).cuda()
            want = _rollout(lib, handle, prompts, n_samples, max_new, 0)
            lib.mtmc_poll_errors(handle)
            got = _rollout(lib, handle, prompts, n_samples, max_new, 1)
            with pytest.raises(lib.MtmcError, match="persistent launch waited longer.*results are right"):
                lib.mtmc_poll_errors(handle)
            again = _rollout(lib, handle, prompts, n_samples, max_new, 10_000_000)
            lib.mtmc_poll_errors(handle)
            for other in (got, again):
                assert all(torch.equal(a, b) for a, b in zip(want, other)), (n_prompts, plen, n_samples, max_new)
    finally:
        lib.mtmc_weights_destroy(handle)


@pytest.mark.parametrize("shape", ["1p5b", "fp32"])
def test_calls_after_one_that_gave_up(lib, shape):
    """16 of them run separate launches, unless the limit is set again."""
    import torch
    cfg, handle = _policy(lib, shape)

    def told():
        got.append([t.cpu() for t in lib.mtmc_rollout(handle, prompts, 2, 6, 1.0, 3)])
        try:
            lib.mtmc_poll_errors(handle)
        except lib.MtmcError as e:
            assert "results are right" in str(e)
            return True
        return False

    try:
        prompts, got = torch.from_numpy(inputs.make_prompts(2, 20, cfg.vocab, seed=1)).cuda(), []
        lib.mtmc_set_option(handle, lib.MTMC_OPT_PERSISTENT_DECODE, 1)
        assert [told() for _ in range(18)] == [True] + 16 * [False] + [True]
        lib.mtmc_set_option(handle, lib.MTMC_OPT_PERSISTENT_DECODE, 1)
        assert [told() for _ in range(2)] == [True, False]
        assert all(torch.equal(a, b) for other in got[1:] for a, b in zip(got[0], other))
    finally:
        lib.mtmc_weights_destroy(handle)


@pytest.mark.parametrize("shape,call", [("1p5b", (2, 100, 2, 12)), ("1p5b", (3, 100, 8, 6)), ("1p5b", (6, 100, 8, 6)),
                                        ("1p5b", (8, 100, 8, 6)), ("7b", (4, 100, 8, 5)), ("fp32", (4, 32, 2, 20))])
@pytest.mark.parametrize("held", [16, 200, 512])  # workgroups of the other kernel; up to two of them share a CU
def test_beside_another_stream(lib, shape, call, held):
    import torch
    cfg, handle = _policy(lib, shape)
    n_prompts, plen, n_samples, max_new = call
    try:
        prompts = torch.from_numpy(inputs.make_prompts(n_prompts, plen, cfg.vocab, seed=plen)).cuda()
        ws = torch.empty(lib.mtmc_rollout_workspace_bytes(handle, *call), dtype=torch.uint8, device="cuda")
        want = _rollout(lib, handle, prompts, n_samples, max_new, 0, workspace=ws)
        out = torch.empty(held * 256, dtype=torch.float32, device="cuda")
        mine, other = torch.cuda.Stream(), torch.cuda.Stream()
        torch.cuda.synchronize()
        for limit in (300, 10_000_000):  # microseconds; the other kernel takes about 13 000
            lib.mtmc_set_option(handle, lib.MTMC_OPT_PERSISTENT_DECODE, limit)
            lib.mtmc_mfma_probe(out, held, 60_000, stream=other)
            with torch.cuda.stream(mine):
                got = lib.mtmc_rollout(handle, prompts, n_samples, max_new, 1.0, 3, workspace=ws, stream=mine)
            torch.cuda.synchronize()
            assert all(torch.equal(a, b.cpu()) for a, b in zip(want, got)), (held, limit)
            try:
                lib.mtmc_poll_errors(handle)
            except lib.MtmcError as e:  # whether the other kernel was in the way is up to the device
                assert limit == 300 and "results are right" in str(e)
    finally:
        lib.mtmc_weights_destroy(handle)


OTHER_PROCESS = """
import sys
import torch
from paper_2511_20100_amd import inputs, mtmc as lib
import test_gpu_persistent_given_up as here
cfg, handle = here._policy(lib, "1p5b")
prompts = torch.from_numpy(inputs.make_prompts(2, 20, cfg.vocab, seed=1)).cuda()
print("ready", flush=True)
for _ in range(20):
    out = here._rollout(lib, handle, prompts, 8, 12, 1)  # a persistent launch would be told of
    lib.mtmc_poll_errors(handle)
torch.save(out, sys.argv[1])
"""


def test_two_processes(lib, tmp_path):
    """The one that came first has the persistent launches, the other one separate ones, at the same time."""
    import os
    import subprocess
    import sys
    import torch
    cfg, handle = _policy(lib, "1p5b")
    try:
        prompts = torch.from_numpy(inputs.make_prompts(2, 20, cfg.vocab, seed=1)).cuda()
        want = _rollout(lib, handle, prompts, 8, 12, 0)
        with pytest.raises(lib.MtmcError, match="results are right"):  # this process has them
            _rollout(lib, handle, prompts, 8, 12, 1)
            lib.mtmc_poll_errors(handle)
        root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
        env = dict(os.environ, PYTHONPATH=os.pathsep.join([root, os.path.join(root, "tests"), os.environ.get("PYTHONPATH", "")]))
        path = str(tmp_path / "out.pt")
        with subprocess.Popen([sys.executable, "-c", OTHER_PROCESS, path], stdout=subprocess.PIPE, text=True, env=env) as other:
            assert other.stdout.readline().strip() == "ready"
            while other.poll() is None:
                got = _rollout(lib, handle, prompts, 8, 12, 10_000_000)
                assert all(torch.equal(a, b) for a, b in zip(want, got))
            assert other.returncode == 0
        lib.mtmc_poll_errors(handle)
        assert all(torch.equal(a, b) for a, b in zip(want, torch.load(path)))
    finally:
        lib.mtmc_weights_destroy(handle)
