"""A dispatch of more 1 KiB units than HIP takes threads in one launch (2^32 at one wave per unit): 33.6 million
tokens of 520 columns (two units each), top-1 on 8 ranks, so that the row kernel's waves stride over a second unit.
About 70 GB of rows. Every packed row is compared with its token's row, bit for bit, on the device; the
combine with weights of one gives x back."""
import pytest
import torch

from paper_2607_06202_amd import epl
from tests.gpu_util import device

pytestmark = pytest.mark.gpu

R, E, H = 8, 8, 520
Tr = (1 << 22) + 1031
T = R * Tr


def test_more_units_than_one_launch_has_waves():
    dev = device()
    if torch.cuda.get_device_properties(dev).total_memory < 200 * 2 ** 30:
        pytest.skip("needs about 110 GB of device memory")
    assert T * 2 * 64 > 1 << 32
    g = torch.Generator(device=dev)
    g.manual_seed(11)
    idx = torch.randint(0, E, (T, 1), generator=g, device=dev, dtype=torch.int32)
    x = torch.empty(T, H, dtype=torch.bfloat16, device=dev)
    step = 1 << 22
    for t0 in range(0, T, step):
        x[t0:t0 + step].normal_(generator=g)
    cfg = epl.config(R, E, 1, H, Tr)
    L, recv, _ = epl.layout_dispatch(cfg, idx, x)
    torch.cuda.synchronize()
    rows = L.pair_row.view(-1)
    assert int(rows.min()) == 0 and int(rows.max()) == T - 1
    xv, rv = x.view(torch.int16), recv.view(torch.int16)
    for t0 in range(0, T, step):
        t1 = min(T, t0 + step)
        assert torch.equal(rv[rows[t0:t1].long()], xv[t0:t1]), "tokens [%d, %d)" % (t0, t1)
    w = torch.ones(T, 1, dtype=torch.float32, device=dev)
    out = epl.combine(cfg, recv, w, L)
    torch.cuda.synchronize()
    for t0 in range(0, T, step):
        t1 = min(T, t0 + step)
        assert torch.equal(out[t0:t1].float(), x[t0:t1].float()), "tokens [%d, %d)" % (t0, t1)
