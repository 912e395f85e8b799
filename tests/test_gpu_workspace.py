"""What a rollout's workspace holds per block of the policy: the keys and values, and the buffers of the one-launch forms only
where a step of the call can take such a form."""
import pytest

pytestmark = pytest.mark.gpu

from paper_2511_20100_amd import inputs

D128 = inputs.ModelConfig(1, 1536, 12, 2, 128, 8960, 272, dtype="bf16")
D64 = inputs.ModelConfig(1, 1536, 24, 4, 64, 8960, 272, dtype="bf16")
F32 = inputs.ModelConfig(1, 256, 4, 2, 64, 688, 272, dtype="fp32")
F32_5 = inputs.ModelConfig(1, 320, 5, 1, 64, 688, 272, dtype="fp32")  # five queries per kv head: does not fit
F32_WIDE = inputs.ModelConfig(1, 1536, 12, 2, 128, 2048, 272, dtype="fp32")


@pytest.mark.parametrize("cfg,call,rows", [
    (D128, (1, 40, 1, 8), 16), (D128, (4, 40, 8, 8), 32), (D128, (8, 40, 8, 8), 64),
    (D128, (1, 40, 1, 1), 0),     # no decode step
    (D128, (16, 40, 8, 8), 0),    # 128 rows
    (D128, (16, 40, 5, 8), 0),    # 80
    (D128, (130, 40, 1, 8), 0),   # 128 and 2, with the splits of 128
    (D64, (1, 40, 1, 8), 0), (D64, (8, 40, 8, 8), 0),
    (F32, (4, 40, 2, 8), 8),
    (F32, (4, 40, 2, 1), 0), (F32, (4, 400, 2, 8), 0), (F32, (128, 40, 1, 8), 0),
    (F32_5, (4, 40, 2, 8), 0), (F32_WIDE, (128, 40, 1, 8), 0),
])
def test_bytes_per_block(cfg, call, rows):
    from paper_2511_20100_amd import mtmc as lib
    n_prompts, plen, n_samples, max_new = call

    def size(layers, ragged):
        c = cfg.with_(n_layers=layers)
        handle = lib.mtmc_weights_create(lib.make_config(c, 1024), inputs.make_weights(c, seed=0).blob())
        try:
            query = lib.mtmc_rollout_ragged_workspace_bytes if ragged else lib.mtmc_rollout_workspace_bytes
            return query(handle, *call)
        finally:
            lib.mtmc_weights_destroy(handle)

    bf = cfg.dtype == "bf16"
    per_group = min(n_prompts, max(1, 128 // n_samples)) if bf else n_prompts
    full, pages = plen // 16, -(-(plen + max_new) // 16)
    n_pages = per_group * full + per_group * n_samples * (pages - full)
    kv = 2 * n_pages * cfg.n_kv_heads * 16 * cfg.head_dim * (2 if bf else 4)
    if bf:
        one_launch = 2 * rows * (2 * cfg.d_model + cfg.d_ffn)
    else:  # three sets
        one_launch = 3 * rows * 4 * (2 * cfg.n_q_heads * cfg.head_dim + 2 * cfg.n_kv_heads * cfg.head_dim + 2 * cfg.d_model + cfg.d_ffn)
    assert abs(size(5, False) - size(1, False) - 4 * (kv + one_launch)) <= 4 * 256
    if cfg is D128 and max_new > 1:  # live rows are packed into 64 slots at most
        grown = size(5, True) - size(1, True) - 4 * 2 * (min(n_prompts, per_group * 4 if n_prompts > per_group else per_group, 128) * full +
                                                         per_group * n_samples * pages) * cfg.n_kv_heads * 16 * cfg.head_dim * 2
        most = min(64, -(-per_group * n_samples // 16) * 16)
        assert abs(grown - 4 * 2 * most * (2 * cfg.d_model + cfg.d_ffn)) <= 4 * 256


WIDE = inputs.ModelConfig(1, 3584, 28, 4, 128, 18944, 272, dtype="bf16")  # 10 gate / up tiles: from 17 rows all hand-overs are counted


@pytest.mark.parametrize("cfg,n_prompts,handed_in_8_splits", [(D128, 4, 1), (D128, 6, 1), (D128, 8, 1), (WIDE, 4, 0)])
def test_no_room_for_hand_overs_that_nobody_asks_for(cfg, n_prompts, handed_in_8_splits):
    from paper_2511_20100_amd import mtmc as lib
    handle = lib.mtmc_weights_create(lib.make_config(cfg, 1024), inputs.make_weights(cfg, seed=0).blob())
    try:
        # the first call decodes nothing: the difference is what the one-launch step takes
        one, two = (lib.mtmc_rollout_workspace_bytes(handle, n_prompts, 40, 8, max_new) for max_new in (1, 2))
    finally:
        lib.mtmc_weights_destroy(handle)
    rows, d, n_qkv = n_prompts * 8, cfg.d_model, (cfg.n_q_heads + 2 * cfg.n_kv_heads) * 128
    taken = 2 * rows * (2 * d + cfg.d_ffn) + 2 * 64 * 256 * 4 + handed_in_8_splits * 4 * rows * (2 * n_qkv + 8 * d)
    assert abs(two - one - taken) <= 16 << 10  # the counters, and the alignment of each buffer
