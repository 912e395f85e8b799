"""The LDS-staged matrix kernels over the sizes at which they choose another tile, at remainders of features, tokens
and vocabulary: a sequence scored alone and in a call of many, and both against the direct kernels.  A block that is
missed, taken twice or read from the wrong place moves logits by their own size."""
import pytest

pytestmark = pytest.mark.gpu

from parity import LOGP_TOL_BF16
from paper_2511_20100_amd import inputs

# 512 / 256 / 1376 features (86 row tiles: remainders of 128, 192 and 256) and 2064 vocabulary entries (129 tiles)
CFG = inputs.ModelConfig(1, 256, 2, 1, 128, 688, 2064, dtype="bf16")
# The forms differ where a value falls on the other side of an fp16 rounding (the direct kernels' silu differs from the
# staged ones' by 1e-6; the row norm of large calls adds its squares in another order than that of small ones).  Each form
# is within LOGP_TOL_BF16 = 1e-2 of the exact value (what fp16 operands give), so that bounds their difference up to a factor
# of two; with one block of layers it is an order smaller, and a wrong block gives differences of order 1.
TOL = LOGP_TOL_BF16


@pytest.fixture(scope="module")
def lib():
    import torch
    from paper_2511_20100_amd import mtmc
    torch.cuda.set_device(0)
    return mtmc


@pytest.fixture(scope="module")
def handle(lib):
    w = inputs.make_weights(CFG, seed=0, std=0.05, gain_std=0.1)
    handle = lib.mtmc_weights_create(lib.make_config(CFG, 512), w.blob())
    yield handle
    lib.mtmc_weights_destroy(handle)


def _lds(lib, handle, on):
    lib.mtmc_set_option(handle, lib.MTMC_OPT_GEMM_LDS_MIN_BLOCKS, 1 if on else 1 << 20)


@pytest.mark.parametrize("n_seqs,seq_len,prompt_len", [(2, 33, 1), (2, 64, 60), (3, 85, 20), (3, 343, 2), (9, 233, 7), (16, 259, 3),
                                                       (47, 128, 64), (63, 190, 90), (129, 257, 250), (260, 257, 200)])
def test_scoring_is_the_same_in_every_tile(lib, handle, n_seqs, seq_len, prompt_len):
    import torch
    seqs = torch.from_numpy(inputs.make_sequences(n_seqs, seq_len, CFG.vocab, seed=4)).cuda()
    _lds(lib, handle, True)
    lp, top1, margin = lib.mtmc_score(handle, seqs, prompt_len, want_top1=True)
    assert torch.equal(lib.mtmc_score(handle, seqs, prompt_len), lp)
    for s in (0, n_seqs - 1):
        one = lib.mtmc_score(handle, seqs[s:s + 1].contiguous(), prompt_len, want_top1=True)
        assert float((one[0][0] - lp[s]).abs().max()) <= TOL and float((one[2][0] - margin[s]).abs().max()) <= 2 * TOL
        clear = margin[s] > 2 * TOL
        assert torch.equal(one[1][0][clear], top1[s][clear])
    _lds(lib, handle, False)
    direct = lib.mtmc_score(handle, seqs, prompt_len)
    lib.mtmc_poll_errors(handle)
    assert float((direct - lp).abs().max()) <= TOL


@pytest.mark.parametrize("n_states,state_len,n_actions,max_len", [(1, 2, 3, 5), (3, 65, 7, 33), (8, 200, 40, 17)])
def test_packed_candidates_are_the_same_in_every_tile(lib, handle, n_states, state_len, n_actions, max_len):
    import torch
    states = torch.from_numpy(inputs.make_prompts(n_states, state_len, CFG.vocab, seed=5)).cuda()
    actions, lens = (torch.from_numpy(x).cuda() for x in inputs.make_actions(n_states, n_actions, max_len, CFG.vocab, 6, 0))
    _lds(lib, handle, True)
    tok, act, _ = lib.mtmc_score_actions(handle, states, actions, lens)
    one = lib.mtmc_score_actions(handle, states[:1].contiguous(), actions[:1].contiguous(), lens[:1].contiguous())
    assert float((one[0][0] - tok[0]).abs().max()) <= TOL
    assert float((one[1][0] - act[0]).abs().max()) <= TOL * max_len
    _lds(lib, handle, False)
    direct = lib.mtmc_score_actions(handle, states, actions, lens)
    lib.mtmc_poll_errors(handle)
    assert float((direct[0] - tok).abs().max()) <= TOL


# q, k and v heads of both sizes, an odd number of them (a wavefront's last pair of 64-dim heads is half empty), sequences
# that end inside a page and blocks that end inside a sequence: the projection that rotates and writes the cache in its
# epilogue, against the separate kernels (few tokens or the direct kernels).
@pytest.mark.parametrize("heads,kv_heads,head_dim", [(3, 1, 64), (4, 4, 64), (3, 1, 128), (12, 2, 128), (8, 8, 64)])
@pytest.mark.parametrize("n_seqs,seq_len", [(8, 129), (1, 1025), (13, 190), (150, 97)])
def test_rotary_epilogue_is_the_separate_kernels(lib, heads, kv_heads, head_dim, n_seqs, seq_len):
    import torch
    cfg = inputs.ModelConfig(2, heads * head_dim, heads, kv_heads, head_dim, 256, 512, dtype="bf16")
    handle = lib.mtmc_weights_create(lib.make_config(cfg, 1280), inputs.make_weights(cfg, seed=1, std=0.04, gain_std=0.1).blob())
    seqs = torch.from_numpy(inputs.make_sequences(n_seqs, seq_len, cfg.vocab, seed=7)).cuda()
    _lds(lib, handle, True)
    lp = lib.mtmc_score(handle, seqs, 1)
    short = lib.mtmc_score(handle, seqs[-1:, :seq_len // 2].contiguous(), 1)
    _lds(lib, handle, False)
    direct = lib.mtmc_score(handle, seqs, 1)
    lib.mtmc_poll_errors(handle)
    lib.mtmc_weights_destroy(handle)
    assert float((direct - lp).abs().max()) <= TOL
    assert float((short[0] - lp[-1, :seq_len // 2 - 1]).abs().max()) <= TOL


def test_wide_projection_between_the_rotary_forms(lib):
    """4608 features x 3584: 1998 tokens are stored by narrower blocks and rotated by the separate kernel, 2997 are rotated in
    the epilogue of 256-feature blocks."""
    import torch
    cfg = inputs.ModelConfig(1, 3584, 28, 4, 128, 256, 512, dtype="bf16")
    handle = lib.mtmc_weights_create(lib.make_config(cfg, 1024), inputs.make_weights(cfg, seed=1, std=0.015, gain_std=0.1).blob())
    try:
        seqs = torch.from_numpy(inputs.make_sequences(3, 1000, cfg.vocab, seed=7))[:, :999].contiguous().cuda()
        _lds(lib, handle, True)
        three, two = lib.mtmc_score(handle, seqs, 1), lib.mtmc_score(handle, seqs[:2].contiguous(), 1)
        _lds(lib, handle, False)
        direct = lib.mtmc_score(handle, seqs, 1)
        lib.mtmc_poll_errors(handle)
        assert float((direct - three).abs().max()) <= TOL and float((two - three[:2]).abs().max()) <= TOL
    finally:
        lib.mtmc_weights_destroy(handle)


# ---- the same bits.  The calls compared below take the same row norm (from 1024 rows on) and the same number of vocabulary
# slices in the LM head (by the scored rows), and split no reduction, so that only what a test is about differs.  (Where the
# reader of a split reduction adds up its slices, no other call runs the same sums in separate launches: the tests above
# bound that form by the tolerance alone.)
def test_scoring_has_the_same_bits_in_every_tile(lib, handle):
    import torch
    seqs = torch.from_numpy(inputs.make_sequences(30, 233, CFG.vocab, seed=4)).cuda()
    _lds(lib, handle, True)
    ref = lib.mtmc_score(handle, seqs, 100)           # 6990 tokens, 3990 scored rows
    for n in (8, 9, 11, 14, 19, 25):                  # from 1864 tokens and 1064 rows
        assert torch.equal(lib.mtmc_score(handle, seqs[:n].contiguous(), 100), ref[:n]), n
    lib.mtmc_poll_errors(handle)


# The samples of a prompt scored as whole sequences, and as candidates of the prompt (packed rows, whose projection is stored and
# rotated by a kernel of its own): 10 880 tokens in one pass, 1196 (on the pages of every eighth row) and 1280 in two.
@pytest.mark.parametrize("heads,kv_heads,head_dim", [(4, 4, 64), (6, 2, 64), (3, 1, 128), (2, 2, 128)])
def test_rotary_epilogue_has_the_bits_of_the_separate_kernels(lib, heads, kv_heads, head_dim):
    import torch
    cfg = inputs.ModelConfig(2, heads * head_dim, heads, kv_heads, head_dim, 688, 1040, dtype="bf16")
    n_states, state_len, n_actions, max_len = 4, 300, 8, 40
    w = inputs.make_weights(cfg, seed=1, std=0.04, gain_std=0.1)
    handle = lib.mtmc_weights_create(lib.make_config(cfg, 1280), w.blob())
    try:
        _lds(lib, handle, True)
        states = torch.from_numpy(inputs.make_prompts(n_states, state_len, cfg.vocab, seed=5)).cuda()
        actions, _ = inputs.make_actions(n_states, n_actions, max_len, cfg.vocab, 6, 0)
        actions = torch.from_numpy(actions).cuda()
        lens = torch.full((n_states, n_actions), max_len, dtype=torch.int32, device="cuda")
        tok = lib.mtmc_score_actions(handle, states, actions, lens)[0]
        whole = torch.cat([states[:, None].expand(-1, n_actions, -1), actions], dim=2).reshape(n_states * n_actions, -1).contiguous()
        lp = lib.mtmc_score(handle, whole, state_len)[:, state_len - 1:].reshape(n_states, n_actions, max_len)
        lib.mtmc_poll_errors(handle)
        assert torch.equal(tok, lp)
    finally:
        lib.mtmc_weights_destroy(handle)


# the epilogue behind a cached prefix: positions that start at 48 and 256, pages of every n_samples-th row, prompts that end
# inside a page, before and behind the last new token of the others
@pytest.mark.parametrize("heads,kv_heads,head_dim", [(4, 4, 64), (3, 1, 128)])
@pytest.mark.parametrize("reuse,max_len,n_samples", [(48, 400, 4), (256, 517, 2)])
def test_rotary_epilogue_behind_a_cached_prefix(lib, heads, kv_heads, head_dim, reuse, max_len, n_samples):
    import torch
    cfg = inputs.ModelConfig(2, heads * head_dim, heads, kv_heads, head_dim, 688, 1040, dtype="bf16")
    handle = lib.mtmc_weights_create(lib.make_config(cfg, 640), inputs.make_weights(cfg, seed=1, std=0.04, gain_std=0.1).blob())
    try:
        _lds(lib, handle, True)
        n = 5  # 1760 and 1305 new tokens
        prompts = torch.from_numpy(inputs.make_prompts(n, max_len, cfg.vocab, seed=2)).cuda()
        lens = torch.tensor([max_len, reuse + 1, max_len - 3, reuse + 16, max_len // 2 + reuse // 2], dtype=torch.int32, device="cuda")
        ws = torch.empty(lib.mtmc_rollout_ragged_workspace_bytes(handle, n, max_len, n_samples, 20), dtype=torch.uint8, device="cuda")
        lib.mtmc_rollout_ragged(handle, prompts, torch.full_like(lens, reuse), n_samples, 20, 1.0, 5, workspace=ws)
        cached = lib.mtmc_rollout_ragged_cached(handle, prompts, lens, n_samples, 20, 1.0, 1, reuse, ws)
        fresh = lib.mtmc_rollout_ragged(handle, prompts, lens, n_samples, 20, 1.0, 1, workspace=torch.empty_like(ws))
        lib.mtmc_poll_errors(handle)
        assert all(torch.equal(a, b) for a, b in zip(cached, fresh))
    finally:
        lib.mtmc_weights_destroy(handle)
