"""epl_layout_dispatch of small layouts (T*k <= 16384 and Tr*k <= 4096), in one launch or with the rows in a
second one, against the CPU oracle, bit for bit, at the edges of the layout's groups: a wave of exactly 64 pairs
and of fewer (k that does not divide 64), one token per group, ragged last groups, few tokens (1 KiB pieces)
and many (4 KiB pieces), the most tokens that are sent in one launch and more, ragged rows, one rank and one choice,
ranks without tokens, 1024 ranks of one expert (beyond the one-launch limit of epl_layout alone), ids at
16-byte alignment and 4 bytes past it. Rows past the valid pairs, and the arrays past them, keep their fill."""
import numpy as np
import pytest
import torch

import oracle
from paper_2607_06202_amd import epl
from paper_2607_06202_amd import workloads as W
from tests.gpu_util import assert_layout_equal, bf16_bits, device, to_dev_bf16

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("R,E,k,Tr,H,payload", [
    (32, 256, 8, 64, 512, "bf16"),      # 16384 pairs: the limit
    (4, 64, 1, 4096, 64, "bf16"),       # top-1, 4096 pairs per rank: groups of 64 tokens, rows in a second launch
    (4, 64, 1, 1024, 1032, "bf16"),     # the most tokens sent in one launch
    (1024, 1024, 1, 16, 72, "bf16"),    # 16384 tokens, in one launch: a group is a whole rank
    (1024, 1024, 2, 8, 128, "fp8"),     # the same, fp8
    (1, 8, 1, 2816, 264, "bf16"),       # one rank and one choice: every lane adds to one word
    (1, 8, 2, 1201, 72, "bf16"),        # one rank, two choices
    (2, 6, 1, 1000, 512, "bf16"),       # two ranks of one choice
    (2, 6, 1, 1025, 3072, "fp8"),       # 2050 tokens of three passes: rows in a second launch
    (1, 4, 1, 4096, 128, "fp8"),        # 4096 tokens on one rank
    (5, 35, 7, 61, 2056, "bf16"),       # 63 of 64 lanes, ragged groups, a second piece of one vector
    (3, 96, 32, 40, 1032, "bf16"),      # two tokens per wave
    (2, 46, 23, 9, 8, "bf16"),          # 46 lanes, one vector per row
    (16, 128, 8, 8, 2048, "bf16"),      # 128 tokens: 1 KiB pieces
    (64, 64, 6, 1, 7168, "bf16"),       # one token per rank
    (1024, 1024, 2, 3, 64, "bf16"),     # 1024 ranks of one expert
    (1, 8, 8, 500, 640, "bf16"),        # one rank: every pair of a token on it
    (16, 64, 8, 30, 2176, "fp8"),       # ragged last pass
    (8, 1024, 20, 40, 128, "fp8"),      # one block per row, 60 of 64 lanes
    (4, 16, 2, 0, 256, "bf16"),         # no tokens
])
@pytest.mark.parametrize("aligned", [True, False])
def test_small_layout_dispatch(R, E, k, Tr, H, payload, aligned):
    dev = device()
    T = R * Tr
    cfg = epl.config(R, E, k, H, Tr, payload)
    assert T * k <= 16384 and Tr * k <= 4096
    seed = 900 + R + k
    idx = W.with_replacement(seed, T, k, -1, E + 1).astype(np.int32)  # duplicates and invalid ids
    x = W.normal_bf16(seed, W.STREAM_X, T * H).reshape(T, H)
    buf = torch.zeros(T * k + 1, dtype=torch.int32, device=dev)
    idx_d = buf[:T * k] if aligned else buf[1:]
    idx_d.copy_(torch.from_numpy(idx).reshape(-1))
    L = epl.alloc_layout(cfg, dev)
    L.recv_src.fill_(-7)
    L.recv_j.fill_(-7)
    recv, sc = epl.alloc_recv(cfg, dev)
    recv.view(torch.uint8).fill_(0xA5)
    epl.layout_dispatch(cfg, idx_d.view(T, k), to_dev_bf16(x, dev), out=L, recv=recv, recv_scale=sc)
    torch.cuda.synchronize()
    ref = oracle.layout(R, E, k, Tr, idx)
    assert_layout_equal(L, ref)
    P = ref.P
    assert (L.recv_src[P:T * k] == -7).all() and (L.recv_j[P:T * k] == -7).all()
    if T == 0:
        return
    if payload == "bf16":
        np.testing.assert_array_equal(bf16_bits(recv[:P]), oracle.dispatch_bf16(x, ref.pair_row, P))
    else:
        q, s = oracle.dispatch_fp8(x, ref.pair_row, P)
        np.testing.assert_array_equal(recv[:P].cpu().numpy(), q)
        np.testing.assert_array_equal(sc[:P].cpu().numpy().view(np.uint32), s.view(np.uint32))
    assert (recv[P:].view(torch.uint8) == 0xA5).all()
