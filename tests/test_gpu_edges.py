"""GPU parity at the edges of tiles, units and launches (run with -m gpu): payload bytes and
reconstruction against the oracle, both bit for bit (the wire format fixes them)."""
import pytest
import torch

from paper_2605_13734_amd import kvgen
from test_gpu_parity import check_contiguous

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("codec", [0, 1])
@pytest.mark.parametrize("group", [32, 64, 128])
@pytest.mark.parametrize("T", [1, 3, 4, 5, 15, 16, 17, 20, 31, 33])
def test_v_metadata_of_short_passes(ref, T, group, codec):
    """Every lane stores the metadata of the rows it finished: passes that end inside its rows."""
    x = kvgen.make_kv(300 + T, 1, 2, 128, T, torch.float16)
    check_contiguous(ref, x, 4, 4, 32, group, codec=codec)
