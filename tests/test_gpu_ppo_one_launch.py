"""The clipped loss as one launch: the workgroup that finds every partial sum tagged adds them up.  A recorded launch has the
same tag at every replay, with new inputs and other calls on the same array between them; from one workgroup to the 128 that
one launch takes, and two launches beyond."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

import mtmc_oracle as oracle
from paper_2511_20100_amd import inputs


@pytest.mark.parametrize("n", [1024, 1025, 65_536, 65_537, 131_072, 131_073])  # 1, 2, 64, 65, 128 and 129 workgroups
def test_replays_of_a_recorded_call(n):
    import torch
    from paper_2511_20100_amd import mtmc
    sets = [inputs.make_ppo_samples(n, seed=s) for s in (1, 2, 3)]
    want = [oracle.ppo_clip_loss(new, old, adv, 0.2) for new, old, adv, _ in sets]
    bufs = [torch.from_numpy(x).cuda() for x in sets[0][:3]]
    out = torch.empty(4, dtype=torch.float64, device="cuda")
    mtmc.mtmc_ppo_clip_loss_static(*bufs, 0.2, out=out)  # looks the array up
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        mtmc.mtmc_ppo_clip_loss_static(*bufs, 0.2, out=out)
    for i in (0, 1, 2, 2, 0):
        for b, x in zip(bufs, sets[i][:3]):
            b.copy_(torch.from_numpy(x))
        out.fill_(float("nan"))
        graph.replay()
        got = out.cpu().numpy()
        assert got[3] == want[i][3] and np.abs(got[:3] - np.array(want[i][:3])).max() <= 1e-9, (i, got, want[i])
        few = mtmc.mtmc_ppo_clip_loss_static(*bufs, 0.2, n=700).cpu().numpy()
        assert np.array_equal(few, mtmc.mtmc_ppo_clip_loss(*[b[:700].contiguous() for b in bufs], 0.2).cpu().numpy())
        assert np.array_equal(got, mtmc.mtmc_ppo_clip_loss(*bufs, 0.2).cpu().numpy())
