"""The decode attention that takes several samples of a prompt in one workgroup (more (sequence, kv head) pairs than CUs):
one to eight query heads per kv head, an even and an odd number of whole prompt pages and none, contexts of one pair of
pages up to several per wavefront, prompts of different lengths.  Every row is replayed on the oracle, and agrees with
the same prompt in a call too small for that form."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

from parity import LOGP_TOL_BF16, check_ragged_by_replay, check_rollout_by_replay
from paper_2511_20100_amd import inputs

MHA8 = inputs.ModelConfig(1, 256, 8, 8, 64, 512, 1040, dtype="bf16")
G2 = inputs.ModelConfig(1, 256, 16, 8, 128, 512, 1040, dtype="bf16")
G4 = inputs.ModelConfig(1, 256, 16, 4, 64, 512, 1040, dtype="bf16")
G7 = inputs.ModelConfig(1, 256, 28, 4, 128, 512, 1040, dtype="bf16")
G4W = inputs.ModelConfig(1, 256, 32, 8, 64, 512, 1040, dtype="bf16")
MHA16 = inputs.ModelConfig(1, 256, 16, 16, 128, 512, 1040, dtype="bf16")


@pytest.fixture(scope="module")
def lib():
    from paper_2511_20100_amd import mtmc
    return mtmc


@pytest.mark.parametrize("name,cfg,n_prompts,plen,n_samples,max_new", [
    # the first two are one round of the plain form
    ("mha-no-whole-page", MHA8, 5, 9, 8, 20),        # 320 pairs; all pages are the sequences' own, 2 of them at the end
    ("mha-odd-pages", MHA8, 5, 55, 8, 12),           # 3 whole pages: two shared, the third taken with the own ones
    ("mha-no-whole-page-four", MHA8, 16, 9, 8, 20),  # the same, four samples per workgroup
    ("mha-odd-pages-four", MHA8, 16, 55, 8, 12),
    ("g4-four", G4W, 9, 70, 12, 40),
    ("mha-eight", MHA16, 16, 21, 8, 9),              # one sequence per wavefront to append for
    ("mha-fifteen-columns", MHA16, 24, 100, 5, 30),
    ("mha-long", MHA8, 8, 330, 6, 6),                # 20 whole pages; two of the six samples per workgroup
    ("g2", G2, 4, 40, 12, 10),
    ("g4", G4, 12, 70, 8, 8),
    ("g7-two-rounds", G7, 16, 37, 8, 8),             # 512 pairs, two sequences per workgroup
], ids=lambda v: v if isinstance(v, str) else None)
def test_samples_in_one_workgroup(lib, name, cfg, n_prompts, plen, n_samples, max_new):
    import torch
    w = inputs.make_weights(cfg, seed=0, std=0.05, gain_std=0.1)
    handle = lib.mtmc_weights_create(lib.make_config(cfg, 512), w.blob())
    try:
        prompts = inputs.make_prompts(n_prompts, plen, cfg.vocab, seed=2)
        last = (n_prompts - 1) * n_samples
        rep = check_rollout_by_replay(handle, w, prompts, n_samples, max_new, 1.0, 1, max_positions=512,
                                      rows=[0, 1, n_samples - 1, n_samples, last, last + n_samples - 1], label=name)
        alone = lib.mtmc_rollout(handle, torch.from_numpy(prompts[-1:]).cuda(), n_samples, max_new, 1.0, 1, seq_offset=last)
        same = (alone[0].cpu().numpy() == rep["ids"][last:]).all(axis=1)
        assert same.any()
        # each is within the tolerance of the exact value
        assert np.abs(alone[1].cpu().numpy() - rep["logprobs"][last:])[same].max() <= 2 * LOGP_TOL_BF16
    finally:
        lib.mtmc_weights_destroy(handle)


def test_prompts_of_different_lengths(lib):
    w = inputs.make_weights(MHA8, seed=0, std=0.05, gain_std=0.1)
    handle = lib.mtmc_weights_create(lib.make_config(MHA8, 512), w.blob())
    try:
        lens = np.array([1, 16, 33, 100, 15, 64, 129, 77, 48, 32], dtype=np.int32)
        prompts = inputs.make_prompts(len(lens), int(lens.max()), MHA8.vocab, seed=2)
        check_ragged_by_replay(handle, w, prompts, lens, 4, 14, 1.0, 1, stop_id=3, max_positions=512, label="ragged")
    finally:
        lib.mtmc_weights_destroy(handle)


@pytest.mark.parametrize("cfg", [G7, MHA8], ids=["g7", "mha8"])
def test_what_a_workspace_held_before_does_not_matter(lib, cfg):
    """Value pages are cleared by the call, key pages are not: every slot a call has not written is masked.  A workspace full
    of NaN patterns gives the bits that a cleared one gives."""
    import torch
    w = inputs.make_weights(cfg, seed=0, std=0.05, gain_std=0.1)
    handle = lib.mtmc_weights_create(lib.make_config(cfg, 256), w.blob())
    try:
        prompts = torch.from_numpy(inputs.make_prompts(9, 53, cfg.vocab, seed=2)).cuda()
        lens = torch.tensor([53, 1, 16, 40, 17, 33, 8, 52, 31], dtype=torch.int32, device="cuda")
        actions, alens = (torch.from_numpy(x).cuda() for x in inputs.make_actions(9, 5, 20, cfg.vocab, 6, 0))
        calls = [
            (lib.mtmc_rollout_workspace_bytes(handle, 9, 53, 8, 21),
             lambda ws: lib.mtmc_rollout(handle, prompts, 8, 21, 1.0, 1, workspace=ws)),
            (lib.mtmc_rollout_ragged_workspace_bytes(handle, 9, 53, 2, 21),
             lambda ws: lib.mtmc_rollout_ragged(handle, prompts, lens, 2, 21, 1.0, 1, workspace=ws)),
            (lib.mtmc_score_workspace_bytes(handle, 9, 53), lambda ws: (lib.mtmc_score(handle, prompts, 5, workspace=ws),)),
            (lib.mtmc_score_actions_workspace_bytes(handle, 9, 53, 5, 20),
             lambda ws: lib.mtmc_score_actions(handle, prompts, actions, alens, workspace=ws)),
        ]
        for n, call in calls:
            got = []
            for fill in (0x00, 0xff):
                ws = torch.full((n,), fill, dtype=torch.uint8, device="cuda")
                got.append([t.clone() for t in call(ws)])
                lib.mtmc_poll_errors(handle)
            assert all(torch.equal(a, b) for a, b in zip(*got))
    finally:
        lib.mtmc_weights_destroy(handle)


@pytest.mark.parametrize("poll", [2, 4])
def test_rows_packed_after_steps_together(lib, poll):
    """Samples of a prompt sit in one workgroup until the first look that frees a tile; from then on every row is alone."""
    cfg = MHA8.with_(vocab=48)
    w = inputs.make_weights(cfg, seed=0, std=0.05, gain_std=0.1)
    handle = lib.mtmc_weights_create(lib.make_config(cfg, 512), w.blob())
    try:
        lib.mtmc_set_option(handle, lib.MTMC_OPT_STOP_POLL_STEPS, poll)
        lens = (3 + np.arange(15) * 11 % 90).astype(np.int32)
        prompts = inputs.make_prompts(len(lens), int(lens.max()), cfg.vocab, seed=2)
        rep = check_ragged_by_replay(handle, w, prompts, lens, 8, 40, 1.0, 1, stop_id=3, max_positions=512, label="packed")
        ends = np.sort(rep["lens"])
        assert (ends < 40).sum() >= 32 and ends[-1] > 4 * poll  # tiles were freed while rows still ran
    finally:
        lib.mtmc_weights_destroy(handle)


@pytest.mark.parametrize("cfg", [MHA8, G7], ids=["mha8", "g7"])
def test_first_batch_of_joining_prompts(lib, cfg):
    """320 sequences through 128 slots: until the batch is packed, the sequences of the first batch get the same bits whether
    the other prompts join it or follow batch after batch, also at sizes where a batch's samples are taken together."""
    import torch
    n_prompts, n_samples, max_new, period = 40, 8, 48, 4
    cfg = cfg.with_(vocab=48)
    w = inputs.make_weights(cfg, seed=0, std=0.05, gain_std=0.1)
    handle = lib.mtmc_weights_create(lib.make_config(cfg, 512), w.blob())
    try:
        lens = torch.from_numpy((30 + np.arange(n_prompts) * 7 % 90).astype(np.int32)).cuda()
        prompts = torch.from_numpy(inputs.make_prompts(n_prompts, int(lens.max()), cfg.vocab, seed=2)).cuda()
        run = lambda stop: [t.cpu() for t in lib.mtmc_rollout_ragged(handle, prompts, lens, n_samples, max_new, 1.0, 1, stop_id=stop)]
        lib.mtmc_set_option(handle, lib.MTMC_OPT_STOP_POLL_STEPS, period)
        joined = run(3)
        lib.mtmc_set_option(handle, lib.MTMC_OPT_ADMIT_PROMPTS, 0)
        lib.mtmc_set_option(handle, lib.MTMC_OPT_STOP_POLL_STEPS, 0)
        lib.mtmc_set_option(handle, lib.MTMC_OPT_HIP_GRAPH, 0)
        free = run(-1)   # without a stop token nothing can join, and samples are taken together
        lib.mtmc_set_option(handle, lib.MTMC_OPT_HIP_GRAPH, 1)
        run(-1)
        static = run(3)  # after a graph of that shape without a stop token
        lib.mtmc_poll_errors(handle)
        # the looks are `period` steps apart, one takes in at most 16 prompts, and the batch is packed one look after the last
        first, steps = 128, period * (-(-(n_prompts - 16) // 16) + 1)
        assert torch.equal(static[0][:first, :steps], joined[0][:first, :steps])
        assert torch.equal(static[1][:first, :steps], joined[1][:first, :steps])
        same = (free[0][:, :4] == static[0][:, :4]).all(dim=1)
        assert (free[1] - static[1])[same][:, :4].abs().max() <= 2 * LOGP_TOL_BF16 and same.float().mean() > 0.5
    finally:
        lib.mtmc_weights_destroy(handle)


@pytest.mark.parametrize("name,cfg,n_prompts,plen,n_samples,max_new", [
    ("mha8", MHA8, 5, 4200, 8, 20),                  # 264 pages: a table of one sequence's own pages for each of two sequences
    ("g7", G7, 14, 1100, 8, 200),
    ("g2", G2, 4, 2300, 9, 12),
], ids=lambda v: v if isinstance(v, str) else None)
def test_equal_lengths_are_mtmc_rollout(lib, name, cfg, n_prompts, plen, n_samples, max_new):
    """Whether a prompt's length is known on the host or on the device only, the same sequences sit in a workgroup."""
    import torch
    w = inputs.make_weights(cfg, seed=0, std=0.05, gain_std=0.1)
    handle = lib.mtmc_weights_create(lib.make_config(cfg, 4352), w.blob())
    try:
        prompts = torch.from_numpy(inputs.make_prompts(n_prompts, plen, cfg.vocab, seed=2)).cuda()
        lens = torch.full((n_prompts,), plen, dtype=torch.int32, device="cuda")
        a = lib.mtmc_rollout(handle, prompts, n_samples, max_new, 1.0, 1)
        b = lib.mtmc_rollout_ragged(handle, prompts, lens, n_samples, max_new, 1.0, 1)
        lib.mtmc_poll_errors(handle)
        assert torch.equal(a[0], b[0]) and torch.equal(a[1], b[1])
    finally:
        lib.mtmc_weights_destroy(handle)


def test_short_prompts_beside_a_long_one(lib):
    """Nearly all pages of the short ones' page-table rows are their own: the table of a workgroup has several hundred entries."""
    w = inputs.make_weights(MHA8, seed=0, std=0.05, gain_std=0.1)
    handle = lib.mtmc_weights_create(lib.make_config(MHA8, 4352), w.blob())
    try:
        lens = np.array([1, 40, 2900, 333, 16], dtype=np.int32)
        prompts = inputs.make_prompts(len(lens), 4200, MHA8.vocab, seed=2)
        check_ragged_by_replay(handle, w, prompts, lens, 8, 40, 1.0, 1, stop_id=-1, max_positions=4352, label="short and long")
    finally:
        lib.mtmc_weights_destroy(handle)
