"""The end of a refresh: the order of the Ritz values, the bf16 copies of the new projectors, made beside the signs or in a
launch of their own."""
import pytest
import torch

from paper_2410_16029_amd import binding as B
from paper_2410_16029_amd import workloads
from test_gpu_parity import DEV

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shapes,r,kw", [
    ([(40, 61), (33, 50), (257, 96)], [20, 32, 33], {}),                   # beside the signs: edges of columns, rows and 256-row runs
    ([(512, 70), (255, 90), (256, 64)], [9, 64, 40], {}),                  # at most 512 rows
    ([(513, 70)], [40], {}),                                               # one more, in few workgroups: apart
    ([(1024, 70), (255, 90), (256, 64)], [9, 64, 40], {}),
    ([(1025, 80)], [40], {}),
    ([(1100, 60), (31, 1200)], [16, 31], {"sides": [B.NG_SIDE_LEFT, B.NG_SIDE_RIGHT]}),    # (right side: 1200 rows)
    ([(1100, 60)] * 20, 17, {}),
    ([(1100, 60)] * 127, 17, {}),                                          # apart, and with one workgroup more beside the signs
    ([(1100, 60)] * 128, 17, {}),
    ([(300, 200)], [70], {"proj_dtype": "bf16"}),
])
def test_bf16_copies_are_the_rounded_projector(shapes, r, kw):
    ls = B.LayerSet(shapes, r, s=2, device=DEV, dtype="bf16", **kw)
    for i in range(len(shapes)):
        ls.buffers[i][B.NG_BUF_AUX].fill_(0x3C)
    rank = [r] * len(shapes) if isinstance(r, int) else r
    ls.refresh(workloads.TorchGradientStream(shapes, min(rank), 0.01, 411, "bf16", DEV).next_set())
    torch.cuda.synchronize()
    assert ls.status() == B.NG_OK
    for i, (a, b) in enumerate(shapes):
        m, k, lay = (b if ls.descs[i].side == 1 else a), rank[i], ls.layouts[i]
        nb, mb = -(-k // 32), -(-m // 32)
        aux = ls.buffers[i][B.NG_BUF_AUX]

        def copy(at, blocks, rows):
            return aux[at:at + 64 * blocks * rows].view(torch.bfloat16).view(blocks, rows, 32).permute(1, 0, 2).reshape(rows, 32 * blocks).float()

        pb, pbt = copy(lay.aux_pb_off, nb, m), copy(lay.aux_pbt_off, mb, k)
        want = ls.P(i).bfloat16().float()
        assert torch.equal(pb[:, :k], want) and torch.equal(pbt[:, :m].T, want)
        assert not bool(pb[:, k:].any()) and not bool(pbt[:, m:].any())


@pytest.mark.parametrize("m,n,r", [(50, 70, 20), (90, 100, 60), (120, 100, 90), (300, 280, 200), (600, 620, 510), (700, 640, 540), (1100, 1070, 1030)])
def test_columns_come_in_the_order_of_their_ritz_values(m, n, r):
    # lanes per value: 32 at order 32, 16, 8, 4, 2, 1; the last beyond 1024
    g = torch.randn(m, n, generator=torch.Generator().manual_seed(5)).to(DEV)
    ls = B.LayerSet([(m, n)], r, s=0, device=DEV, dtype="f32")
    ls.refresh([g])
    torch.cuda.synchronize()
    e = (ls.P(0).double().T @ g.double()).square().sum(1).sqrt()
    # the fp32 gradient products behind the Ritz values have errors of about 1e-6 of the largest, the last
    # orthonormalisation moves the columns by about as much: 20 times that
    assert bool((e[1:] <= e[:-1] + 2e-5 * e[0]).all())
