"""The plain bf16 dispatch (epl_dispatch) at the edges of its 1 KiB units, bit for bit against the CPU
oracle's layout: one and two choices (the kernel with more waves) and three, rows of one vector, of one
unit exactly, of one vector more, and of an odd number of units, with a row pitch, an odd number of
waves, duplicate and invalid ids. Rows past the valid pairs and the gaps between rows keep their fill."""
import numpy as np
import pytest
import torch

import oracle
from paper_2607_06202_amd import epl
from paper_2607_06202_amd import workloads as W
from tests.gpu_util import device, to_dev_bf16

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("k", [1, 2, 3])
@pytest.mark.parametrize("H,pitch", [(8, 64), (512, 0), (520, 576), (1544, 1600)])
def test_plain_dispatch_units(k, H, pitch):
    dev = device()
    R, E, Tr = 3, 24, 67
    T = R * Tr
    cfg = epl.config(R, E, k, H, Tr, "bf16", pitch)
    idx = W.with_replacement(40 + k, T, k, -1, E + 1).astype(np.int32)
    x = W.normal_bf16(40 + k, W.STREAM_X, T * H).reshape(T, H)
    L = epl.layout(cfg, torch.from_numpy(idx).to(dev))
    full = torch.full((T * k, cfg.pitch), -7, dtype=torch.int16, device=dev)
    epl.dispatch(cfg, to_dev_bf16(x, dev), L, full.view(torch.bfloat16)[:, :H])
    torch.cuda.synchronize()
    ref = oracle.layout(R, E, k, Tr, idx)
    got = full.cpu().numpy().view(np.uint16)
    np.testing.assert_array_equal(got[:ref.P, :H], oracle.dispatch_bf16(x, ref.pair_row, ref.P))
    assert (got[ref.P:] == 0xFFF9).all() and (got[:, H:] == 0xFFF9).all()
