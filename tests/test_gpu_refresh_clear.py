"""A refresh clears the history ring and the Gram block, beside whichever of its launches leave room for that: the small
factors (orders up to 32), the factors, the Jacobi's rounds, or in a launch of its own."""
import pytest
import torch

from paper_2410_16029_amd import binding as B
from paper_2410_16029_amd import workloads
from test_gpu_parity import DEV

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shapes,r,s,kw", [
    ([(40, 61), (64, 33), (90, 35)], 20, 4, {}),                               # beside factors of one block
    ([(300, 417), (150, 2330), (131, 140)], 100, 3, {"dtype": "bf16"}),        # beside the factors; a state in column panels
    ([(300, 417), (270, 290)], 250, 0, {}),                                    # no history: the scratch slot
    ([(140, 150)] * 129 + [(141, 133)], 120, 2, {"dtype": "bf16", "hist_dtype": "bf16"}),   # beside the rounds, 520 visits
    ([(330, 350), (400, 417)], 300, 5, {"power_iters": 0}),                    # beside the rounds, order above 256
    ([(140, 150)] * 3, 120, 2, {"sweeps": 1, "power_iters": 0}),
    ([(64, 9001)], 20, 4, {}),                                                 # one matrix, over all workgroups
    ([(40, 61)] * 70 + [(64, 9001)] + [(40, 61)] * 70, 20, 3, {"dtype": "bf16"}),   # a wide one among more than 64
    ([(140, 150)] * 65 + [(150, 4097)] + [(141, 133)], 120, 2, {"dtype": "bf16", "hist_dtype": "bf16"}),
    ([(140, 150)] * 64 + [(150, 4097)] + [(140, 150)] * 64, 120, 2, {}),       # beside the rounds
    ([(130, 140)] * 383, 128, 1, {}),                                          # no room: 1536 visits
])
def test_refresh_leaves_no_history(shapes, r, s, kw):
    kw = dict({"dtype": "f32"}, **kw)
    stream = workloads.TorchGradientStream(shapes, min(r, 100), 0.01, 401, kw["dtype"], DEV)
    ls = B.LayerSet(shapes, r, s=s, device=DEV, **kw)
    for i in range(len(shapes)):
        for b in (B.NG_BUF_H, B.NG_BUF_K):
            ls.buffers[i][b].fill_(0x3C)
    ls.refresh(stream.next_set())
    torch.cuda.synchronize()
    assert ls.status() in (B.NG_OK, B.NG_ERR_NOT_CONVERGED)
    for i in range(len(shapes)):
        for b in (B.NG_BUF_H, B.NG_BUF_K):
            n = ls.sizes[i][b]                       # (buffers are at least 16 bytes long)
            assert not bool(ls.buffers[i][b][:n].any()), (i, b)
