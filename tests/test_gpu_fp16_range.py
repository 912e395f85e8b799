"""Where the fp16 range of a SwiGLU product ends: 65504 is stored and reported by nobody, 65512 rounds to 65504 and is
reported, by the staged and the direct kernels of the scoring pass and by the decode kernels alike."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

from paper_2511_20100_amd import inputs

CFG = inputs.ModelConfig(1, 256, 2, 1, 128, 256, 512, dtype="bf16")


@pytest.fixture(scope="module")
def lib():
    from paper_2511_20100_amd import mtmc
    return mtmc


# gate = 256 (its silu is 256 in fp32), up = 255 + this, all exact: every normalised activation is 1 (the embeddings are +1,
# the attention adds nothing) and a weight row holds its sum in one or two entries
@pytest.mark.parametrize("extra,reported", [(0.875, False), (0.90625, True)])
def test_the_last_value_that_fits(lib, extra, reported):
    import torch
    w = inputs.make_weights(CFG, seed=0, std=0.02)
    zero = lambda name: np.zeros_like(inputs.bf16_bits_to_f32(w.tensors[name]))
    for name in ("layers.0.wo", "layers.0.wdown"):
        w.tensors[name] = inputs.f32_to_bf16_bits(zero(name))
    w.tensors["embed"] = inputs.f32_to_bf16_bits(zero("embed") + 1.0)
    gate, up = zero("layers.0.wgate"), zero("layers.0.wup")
    gate[77, 3] = 256.0
    up[77, 5], up[77, 200] = 255.0, extra
    w.tensors["layers.0.wgate"], w.tensors["layers.0.wup"] = inputs.f32_to_bf16_bits(gate), inputs.f32_to_bf16_bits(up)
    w.drop_cache()
    handle = lib.mtmc_weights_create(lib.make_config(CFG, 64), w.blob())
    try:
        seqs = torch.from_numpy(inputs.make_sequences(3, 40, CFG.vocab, seed=4)).cuda()

        def check():
            if reported:
                with pytest.raises(lib.MtmcError, match="fp16 range"):
                    lib.mtmc_poll_errors(handle)
            else:
                lib.mtmc_poll_errors(handle)

        for min_blocks in (1, 1 << 20):
            lib.mtmc_set_option(handle, lib.MTMC_OPT_GEMM_LDS_MIN_BLOCKS, min_blocks)
            lib.mtmc_score(handle, seqs, 8)
            check()
        for rows in (1, 40, 100):  # the decode steps' kernels: the prompt of one token is prefilled by the direct kernel
            lib.mtmc_rollout(handle, seqs[:1, :1].contiguous(), rows, 3, 1.0, 1)
            check()
    finally:
        lib.mtmc_weights_destroy(handle)
