"""Log-probabilities of a policy that is sure of its next token, from every LM head that leaves one.

After token t the policy gives token t + 1 a logit L of 35 to 65 and every other token one of at most about 15, so the exact
log-probability lies in (-1e-5, 0] for L >= 27 above the rest and rounds to zero: the sum of exponentials, taken relative
to the largest logit, is 1 to within n 2^-24 (n = 2 or 3 roundings of terms and rescalings near 1), its logarithm at most
4e-7 in magnitude, and L plus that is L itself from L = 8 on, where half a unit in the last place is 4.8e-7.  A sum that is
off by a factor (a reference that is not the largest logit itself) shows as multiples of 3.8e-6 of either sign."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

from paper_2511_20100_amd import inputs


@pytest.fixture(scope="module")
def lib():
    from paper_2511_20100_amd import mtmc
    return mtmc


def _sure_weights(d, heads, vocab):
    """The LM-head row of token v is a multiple of the embedding of token v - 1; the blocks add little to it."""
    cfg = inputs.ModelConfig(1, d, heads, 2 if heads > 8 else 1, 128, 256, vocab, dtype="bf16")
    w = inputs.make_weights(cfg, seed=0, std=0.005)
    rng = np.random.default_rng(3)
    embed = inputs.bf16_bits_to_f32(inputs.f32_to_bf16_bits(rng.standard_normal((vocab, d), dtype=np.float32)))
    level = rng.uniform(40.0, 60.0, vocab).astype(np.float32)  # the embeddings' norms add some 10 % to either side
    w.tensors["embed"] = inputs.f32_to_bf16_bits(embed)
    w.tensors["lm_head"] = inputs.f32_to_bf16_bits(np.roll(embed, 1, axis=0) * (level / d)[:, None])
    w.drop_cache()
    return cfg, w


def _walk(n, length, vocab):
    return ((np.arange(n)[:, None] * 977 + np.arange(length)) % vocab).astype(np.int32)


@pytest.mark.parametrize("n_seqs,seq_len", [(1, 40), (9, 130), (33, 150)])  # one block of rows, narrow blocks, both widths
def test_scoring(lib, n_seqs, seq_len):
    import torch
    cfg, w = _sure_weights(512, 4, 4112)
    handle = lib.mtmc_weights_create(lib.make_config(cfg, 256), w.blob())
    try:
        seqs = torch.from_numpy(_walk(n_seqs, seq_len, cfg.vocab)).cuda()
        for min_blocks in (1, 1 << 20):
            lib.mtmc_set_option(handle, lib.MTMC_OPT_GEMM_LDS_MIN_BLOCKS, min_blocks)
            lp, top1, margin = lib.mtmc_score(handle, seqs, 1, want_top1=True)
            plain = lib.mtmc_score(handle, seqs, 1)
            lib.mtmc_poll_errors(handle)
            assert torch.equal(top1, seqs[:, 1:]) and float(margin.min()) > 20.0
            assert float(lp.abs().max()) == 0.0 and float(plain.abs().max()) == 0.0, min_blocks
    finally:
        lib.mtmc_weights_destroy(handle)


# the general sampling head, the persistent one of up to 64 rows (widths it is built for), the forms of 65 to 128 rows
@pytest.mark.parametrize("d,heads,vocab,rows", [(256, 2, 4112, 40), (512, 4, 4112, 5), (512, 4, 4112, 60), (1536, 12, 33008, 3), (1536, 12, 33008, 64),
                                                (512, 4, 4112, 100), (512, 4, 33008, 100)])
def test_sampling(lib, d, heads, vocab, rows):
    import torch
    cfg, w = _sure_weights(d, heads, vocab)
    handle = lib.mtmc_weights_create(lib.make_config(cfg, 128), w.blob())
    try:
        walk = _walk(rows, 20, cfg.vocab)
        prompts = torch.from_numpy(walk[:, :8].copy()).cuda()
        for temperature in (1.0, 0.0):
            ids, lp = lib.mtmc_rollout(handle, prompts, 1, 12, temperature, 1)
            lib.mtmc_poll_errors(handle)
            assert np.array_equal(ids.cpu().numpy(), walk[:, 8:])
            assert float(lp.abs().max()) == 0.0
    finally:
        lib.mtmc_weights_destroy(handle)
