"""The one-launch kernels at the edges of their work units, against the CPU oracle, bit for bit (the
outputs are copies, whole numbers and an fmaf chain of fixed order, so no tolerance): send batches of one
to four tokens whose last is short, waves without a unit, a wave's units in one and in several groups of
loads, one and several 1 KiB chunks per combine task with a short last task, and choices that fill one,
or run past one, group of gathers; layers whose
senders go on to combine and layers that have workgroups for it."""
import pytest

from paper_2607_06202_amd import epl
from tests.test_gpu_data_as_flag import _layer as daf_layer
from tests.test_gpu_decomposed import _check as decomposed_layer
from tests.test_gpu_sentinel import _layer as sentinel_layer

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("path", ["decomposed", "sentinel", "flag", "checksum"])
@pytest.mark.parametrize("R,E,k,Tr,H,seed", [
    (1, 4, 1, 1, 8, 0),          # one token of one vector: three waves without a unit
    (3, 6, 2, 7, 512, 1),        # 21 tokens, one chunk each
    (2, 8, 8, 257, 1024, 2),     # 514 tokens: two per batch, the last batch whole
    (7, 28, 9, 149, 520, 3),     # 1,043 tokens, ragged rows, a second group of one gather
    (16, 16, 4, 641, 264, 4),    # 10,256 tokens: two rounds of batches of four, half a chunk
    (8, 32, 16, 33, 2568, 5),    # two whole groups of gathers, six chunks, the last of one vector
    (8, 64, 3, 513, 3592, 6),    # 4,104 tokens of eight chunks: several chunks per task
    (5, 40, 25, 11, 7168, 7),    # 55 tokens of 14 chunks: four groups of loads per wave
    (16, 64, 2, 400, 1032, 8),   # 6,400 tokens, two choices: two rounds of batches, three chunks
    (8, 32, 1, 1500, 264, 9),    # 12,000 tokens, one choice, half a chunk: combined by workgroups of their own
    (32, 64, 3, 64, 4104, 10),   # 2,048 tokens of nine chunks
])
def test_units(path, R, E, k, Tr, H, seed):
    if path == "decomposed":
        decomposed_layer(R, E, k, Tr, H, seed)
    elif path == "sentinel":
        sentinel_layer(R, E, k, Tr, H, seed)
    else:
        variant = epl.DAF_TOKEN_FLAG_FUSION if path == "flag" else epl.DAF_DATA_CHECKSUM
        daf_layer(variant, R, E, k, Tr, H, seed, epoch=1)
