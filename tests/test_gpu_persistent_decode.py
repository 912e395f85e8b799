"""Decode steps of up to 64 rows as one persistent launch: the bits of the separate launches, at every split of the work that
the launch knows (gate / up tiles per workgroup, ranges of the down projection, context chunks, one to four row tiles of the
QKV projection per workgroup, one to four tiles of rows), from one row to full tiles, with empty slots, from two threads, and
with a wait that gives up."""
import threading

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

from paper_2511_20100_amd import inputs

V = 1040
SHAPES = {
    # gate / up: 4 tiles per workgroup; down: one split of 8 ranges
    "narrow": inputs.ModelConfig(3, 1536, 12, 2, 128, 512, V, dtype="bf16"),
    # 6 and 2 tiles; 8 splits of 5 ranges
    "1p5b": inputs.POLICY_1P5B.with_(n_layers=2, vocab=V),
    # 10 tiles, two QKV tiles per workgroup; splits of 4 ranges
    "7b": inputs.POLICY_7B.with_(n_layers=1, vocab=V),
    # 4 and 2 tiles, one kv head per query head; 4 splits of 8 ranges
    "mha": inputs.POLICY_1P3B_MHA.with_(n_layers=2, vocab=V),
    # fewer context chunks, a padded feed-forward width
    "wide-kv": inputs.ModelConfig(2, 1600, 16, 8, 128, 1104, V, dtype="bf16"),
}


@pytest.fixture(scope="module")
def lib():
    from paper_2511_20100_amd import mtmc
    return mtmc


@pytest.fixture(scope="module", params=SHAPES)
def policy(request, lib):
    cfg = SHAPES[request.param]
    handle = lib.mtmc_weights_create(lib.make_config(cfg, 2400), inputs.make_weights(cfg, seed=0, std=0.04, gain_std=0.1).blob())
    yield cfg, handle
    lib.mtmc_weights_destroy(handle)


def _both(lib, handle, call):
    """call() as separate launches and as persistent ones; the latter must really have run (a wait of a microsecond stalls)."""
    import torch
    got = []
    for value in (0, 10_000_000):
        lib.mtmc_set_option(handle, lib.MTMC_OPT_PERSISTENT_DECODE, value)
        got.append([t.cpu() for t in call()])
        lib.mtmc_poll_errors(handle)
    lib.mtmc_set_option(handle, lib.MTMC_OPT_PERSISTENT_DECODE, 1)
    try:
        call()
        with pytest.raises(lib.MtmcError, match="persistent"):
            lib.mtmc_poll_errors(handle)
    finally:
        lib.mtmc_set_option(handle, lib.MTMC_OPT_PERSISTENT_DECODE, 10_000_000)
    got.append([t.cpu() for t in call()])  # nothing is left of the stalled call
    lib.mtmc_poll_errors(handle)
    torch.cuda.synchronize()
    for other in got[1:]:
        assert all(torch.equal(a, b) for a, b in zip(got[0], other))
    assert torch.isfinite(got[0][1]).all()


@pytest.mark.parametrize("n_prompts,plen,n_samples,max_new", [
    (1, 1, 1, 20),     # one page, then two; one context chunk
    (1, 127, 1, 4),    # two chunks
    (1, 300, 2, 20),   # three to five; across a page
    (2, 1100, 1, 5),   # eight
    (5, 90, 3, 40),    # a full tile but for one row
    (2, 700, 8, 18),   # a full tile
])
def test_the_bits_of_separate_launches(lib, policy, n_prompts, plen, n_samples, max_new):
    import torch
    cfg, handle = policy
    prompts = torch.from_numpy(inputs.make_prompts(n_prompts, plen, cfg.vocab, seed=plen)).cuda()
    _both(lib, handle, lambda: lib.mtmc_rollout(handle, prompts, n_samples, max_new, 1.0, 3))


# more than one tile of rows: which shapes that form takes, and where its units are more than one round
MANY_ROWS = {
    "1p5b": SHAPES["1p5b"],
    "7 blocks": inputs.POLICY_1P5B.with_(n_layers=7, vocab=V),                      # more than the buffers that rows of qkv take in turn
    "7b": SHAPES["7b"],                                                             # up to 32 rows
    "qkv-2-rounds": inputs.ModelConfig(2, 1536, 24, 4, 128, 8960, V, dtype="bf16"),  # 512 units of 16 ranges
    "qkv-3-rounds": inputs.ModelConfig(2, 1536, 28, 4, 128, 8960, V, dtype="bf16"),  # 576 units of 8 ranges
}


@pytest.mark.parametrize("shape,calls", [
    ("1p5b", [(3, 1, 6, 18), (17, 1100, 1, 5), (2, 2300, 9, 4), (4, 300, 8, 20),   # 18, 17, 18, 32 rows: 1, 3, 3, 2 chunks
              (11, 127, 3, 4), (5, 700, 8, 18), (6, 20, 8, 12),                     # 33, 40, 48 rows
              (7, 90, 7, 20), (8, 300, 8, 20), (4, 1500, 16, 3)]),                  # 49, 64, 64 rows
    ("7 blocks", [(17, 40, 1, 9), (4, 300, 8, 6), (6, 700, 8, 6), (8, 20, 8, 9)]),  # 17, 32, 48, 64 rows
    ("7b", [(17, 300, 1, 6), (4, 100, 8, 12), (3, 1500, 8, 4)]),
    ("qkv-2-rounds", [(3, 40, 8, 6), (5, 140, 8, 6), (8, 40, 8, 6)]),
    ("qkv-3-rounds", [(3, 40, 8, 6), (5, 140, 8, 6), (8, 40, 8, 6)]),
])
def test_the_bits_with_several_tiles_of_rows(lib, shape, calls):
    import torch
    cfg = MANY_ROWS[shape]
    handle = lib.mtmc_weights_create(lib.make_config(cfg, 2400), inputs.make_weights(cfg, seed=0, std=0.04, gain_std=0.1).blob())
    try:
        for n_prompts, plen, n_samples, max_new in calls:
            prompts = torch.from_numpy(inputs.make_prompts(n_prompts, plen, cfg.vocab, seed=plen)).cuda()
            _both(lib, handle, lambda: lib.mtmc_rollout(handle, prompts, n_samples, max_new, 1.0, 3))
    finally:
        lib.mtmc_weights_destroy(handle)


def test_lengths_stop_tokens_and_empty_slots(lib, policy):
    """Prompts of different lengths; sequences end, the rest is packed into fewer tiles (from 24 rows, from 64 and from 160)."""
    import torch
    cfg, handle = policy
    for n_prompts, n_samples, max_new in ((3, 8, 24), (8, 8, 24), (20, 8, 24)):
        lens = torch.from_numpy(np.random.default_rng(n_prompts).integers(1, 90, n_prompts).astype(np.int32)).cuda()
        prompts = torch.from_numpy(inputs.make_prompts(n_prompts, 90, cfg.vocab, seed=5)).cuda()
        free = lib.mtmc_rollout_ragged(handle, prompts, lens, n_samples, max_new, 1.0, 4)[0].cpu().numpy()
        # a stop token that ends sequences early and leaves a few to the end
        ends = {t: (free == t).any(axis=1).sum() for t in np.unique(free[:, :8])}
        stop = int(max(ends, key=ends.get))
        lib.mtmc_set_option(handle, lib.MTMC_OPT_STOP_POLL_STEPS, 2)
        outs = []
        for value in (0, 10_000_000):
            lib.mtmc_set_option(handle, lib.MTMC_OPT_PERSISTENT_DECODE, value)
            outs.append([t.cpu() for t in lib.mtmc_rollout_ragged(handle, prompts, lens, n_samples, max_new, 1.0, 4, stop_id=stop)])
            lib.mtmc_poll_errors(handle)
        lib.mtmc_set_option(handle, lib.MTMC_OPT_STOP_POLL_STEPS, lib.MTMC_STOP_POLL_CHOOSE)
        assert all(torch.equal(a, b) for a, b in zip(*outs))


def test_two_threads_and_two_handles(lib):
    """Only one call at a time gets the device for persistent launches; whoever does not, gives the same bits."""
    import torch
    cfg = SHAPES["narrow"]
    handles = [lib.mtmc_weights_create(lib.make_config(cfg, 256), inputs.make_weights(cfg, seed=s, std=0.04).blob()) for s in (0, 1)]
    try:
        prompts = torch.from_numpy(inputs.make_prompts(2, 70, cfg.vocab, seed=1)).cuda()
        wss = [torch.empty(lib.mtmc_rollout_workspace_bytes(handles[0], 2, 70, 4, 30), dtype=torch.uint8, device="cuda") for _ in range(3)]
        streams = [torch.cuda.Stream() for _ in range(3)]
        ref = {}
        for h in (0, 1):
            lib.mtmc_set_option(handles[h], lib.MTMC_OPT_PERSISTENT_DECODE, 0)
            for seed in range(6):
                ref[h, seed] = [t.cpu() for t in lib.mtmc_rollout(handles[h], prompts, 4, 30, 1.0, seed)]
            lib.mtmc_set_option(handles[h], lib.MTMC_OPT_PERSISTENT_DECODE, 10_000_000)
        torch.cuda.synchronize()
        got, failed = {}, []

        def work(i):
            try:
                with torch.cuda.stream(streams[i]):
                    for seed in range(6):
                        got[i, seed] = lib.mtmc_rollout(handles[i % 2], prompts, 4, 30, 1.0, seed, workspace=wss[i], stream=streams[i])
            except Exception as e:  # noqa: BLE001  (reported by the test's own thread)
                failed.append(e)

        threads = [threading.Thread(target=work, args=(i,)) for i in range(3)]
        for t in threads:
            t.start()
        for t in threads:
            t.join()
        torch.cuda.synchronize()
        assert not failed, failed
        for h in handles:
            lib.mtmc_poll_errors(h)
        for (i, seed), out in got.items():
            assert all(torch.equal(a, b.cpu()) for a, b in zip(ref[i % 2, seed], out)), (i, seed)
    finally:
        for h in handles:
            lib.mtmc_weights_destroy(h)
