"""Sums of split-K slices by the kernels that read them: one prompt of sizes that leave 2 to 8 slices, widths of one and two chunks per
thread of the norm, against the whole reduction in one block.  That a slice is left out, read twice or misplaced would show here; the order
of the sums, on which their bits hang, is checked by test_slices.py."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

from paper_2511_20100_amd import inputs

V = 1040


@pytest.mark.parametrize("d,heads,kv,ffn", [(1536, 12, 2, 8960), (2080, 16, 2, 2048), (4096, 32, 8, 4096)])
@pytest.mark.parametrize("length", [33, 129, 300, 511])
def test_scores_of_one_sequence(d, heads, kv, ffn, length):
    import torch
    from paper_2511_20100_amd import mtmc as lib
    cfg = inputs.ModelConfig(2, d, heads, kv, 128, ffn, V, dtype="bf16")
    handle = lib.mtmc_weights_create(lib.make_config(cfg, 512), inputs.make_weights(cfg, seed=0, std=0.02, gain_std=0.1).blob())
    try:
        seqs = torch.from_numpy(inputs.make_prompts(1, length, V, seed=length)).cuda()
        got = lib.mtmc_score(handle, seqs, 1).cpu().numpy()
        # the sequence eight times: wider passes, whose products come in other numbers of slices or in none
        many = lib.mtmc_score(handle, seqs.repeat(8, 1).contiguous(), 1).cpu().numpy()
        lib.mtmc_poll_errors(handle)
        # sums in another order move an fp16 operand by an ulp here and there: as the parity tests of this path allow
        assert np.isfinite(got).all() and np.abs(got[0] - many[5]).max() <= 1e-2
    finally:
        lib.mtmc_weights_destroy(handle)
