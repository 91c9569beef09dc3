"""epl_layout_dispatch in three launches (counts, placement, rows: layouts of more than 16384 pairs, of at
most 512 chunks and 256 experts, whose 16-bit sums fit) against the CPU oracle, bit for bit, at the edges of its
count matrix: odd and small numbers of experts (rows of counts that end inside a 16-byte load), a last group of
fewer than four chunks, source ranks whose first chunk lies inside a group, layouts whose chunks are made longer
so that at most 256 of them are launched, a second batch of group rows (more than 256 chunks launched), a single
source rank, chunks of more than 256 pairs (more steps per wave), k that does not divide 64, every pair on one
expert up to the largest 16-bit sums (61440) and one token more (the general path), ids 4 bytes past 16-byte
alignment; fp8 rows."""
import numpy as np
import pytest
import torch

import oracle
from paper_2607_06202_amd import epl
from paper_2607_06202_amd import workloads as W
from tests.gpu_util import assert_layout_equal, bf16_bits, device, to_dev_bf16

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("R,E,k,Tr,payload,routing", [
    (1, 7, 3, 6000, "bf16", "any"),       # one rank, odd E: a row of counts is one short load
    (3, 255, 5, 1111, "bf16", "any"),     # odd E, ragged chunks, ranks starting inside a group
    (24, 192, 8, 128, "bf16", "any"),     # 264 chunks: 240 longer ones are taken
    (130, 130, 8, 16, "bf16", "any"),     # one chunk per rank, a last group of two
    (16, 256, 22, 100, "bf16", "any"),    # k that does not divide 64
    (8, 64, 1, 3000, "bf16", "any"),      # top-1
    (2, 16, 8, 8192, "bf16", "one"),      # all pairs on one expert, 512 pairs per chunk
    (1, 256, 8, 32640, "bf16", "one"),    # 255 chunks of 1024 pairs, all on one expert
    (64, 256, 8, 512, "bf16", "any"),     # 256 chunks of 1024 pairs
    (1, 256, 8, 40000, "bf16", "any"),    # 313 chunks of 1024 pairs: a second batch, partly filled
    (1, 256, 8, 61440, "bf16", "one"),    # 480 chunks of 1024 pairs on one expert: sums of 61440
    (1, 256, 8, 61441, "bf16", "one"),    # 481 chunks: the general path
    (241, 241, 8, 130, "bf16", "any"),    # two chunks per rank, of 128 and 2 tokens
    (249, 249, 8, 193, "fp8", "one"),     # 498 chunks, of 128 and 65 tokens by turns, all on one expert
    (300, 300, 4, 20, "bf16", "any"),     # more than 256 experts: the general path
    (5, 40, 7, 700, "fp8", "any"),
    (256, 256, 8, 40, "fp8", "any"),
])
@pytest.mark.parametrize("aligned", [True, False])
def test_three_launch_layout_dispatch(R, E, k, Tr, payload, routing, aligned):
    dev = device()
    H = 128
    T = R * Tr
    assert T * k > 16384 or Tr * k > 4096
    cfg = epl.config(R, E, k, H, Tr, payload)
    seed = 500 + R + E
    if routing == "one":
        idx = np.full((T, k), E - 1, np.int32)
    else:
        idx = W.with_replacement(seed, T, k, -1, E + 1).astype(np.int32)  # duplicates and invalid ids
    x = W.normal_bf16(seed, W.STREAM_X, T * H).reshape(T, H)
    buf = torch.zeros(T * k + 1, dtype=torch.int32, device=dev)
    idx_d = buf[:T * k] if aligned else buf[1:]
    idx_d.copy_(torch.from_numpy(idx).reshape(-1))
    L = epl.alloc_layout(cfg, dev)
    L.workspace.fill_(0x5A)  # its contents on entry do not matter
    L.recv_src.fill_(-7)
    L.recv_j.fill_(-7)
    recv, sc = epl.alloc_recv(cfg, dev)
    recv.view(torch.uint8).fill_(0xA5)
    epl.layout_dispatch(cfg, idx_d.view(T, k), to_dev_bf16(x, dev), out=L, recv=recv, recv_scale=sc)
    torch.cuda.synchronize()
    ref = oracle.layout(R, E, k, Tr, idx)
    assert_layout_equal(L, ref)
    P = ref.P
    assert (L.recv_src[P:] == -7).all() and (L.recv_j[P:] == -7).all()
    if payload == "bf16":
        np.testing.assert_array_equal(bf16_bits(recv[:P]), oracle.dispatch_bf16(x, ref.pair_row, P))
    else:
        q, s = oracle.dispatch_fp8(x, ref.pair_row, P)
        np.testing.assert_array_equal(recv[:P].cpu().numpy(), q)
        np.testing.assert_array_equal(sc[:P].cpu().numpy().view(np.uint32), s.view(np.uint32))
    assert (recv[P:].view(torch.uint8) == 0xA5).all()
