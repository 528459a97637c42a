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


def _codes_as_values(codes):
    """V rows whose 8-bit codes are exactly `codes` ([T, 128] integers): every group of 32 holds a 0 and a 255,
    so scale = 1 and zero = 0."""
    v = codes.clone()
    v[:, 0::32], v[:, 1::32] = 0, 255
    return v.half()


@pytest.mark.parametrize("kind", ["equal", "one", "two", "powers", "fibonacci", "squares", "steps"])
def test_code_construction(ref, kind):
    """Byte histograms that take the join through its corners: all weights equal (256 leaves in one round), one
    or two heavy symbols, a node per round, ties between leaves and joined nodes, odd ones out."""
    T, g = 4 * 128, torch.Generator().manual_seed(11)
    n = 256
    if kind == "equal":
        w = torch.ones(n)
    elif kind == "one":
        w = torch.zeros(n)
        w[77] = 1
    elif kind == "two":
        w = torch.zeros(n)
        w[5], w[6] = 1, 2
    elif kind == "powers":
        w = 2.0 ** -(torch.arange(n) % 24).double()
    elif kind == "fibonacci":
        w = 1.618 ** -(torch.arange(n) % 20).double()
    elif kind == "squares":
        w = (torch.arange(n).double() + 1) ** -2
    else:
        w = (1 + torch.arange(n) // 37).double()
    codes = torch.multinomial(w.double(), T * 128, replacement=True, generator=g).reshape(T, 128)
    x = kvgen.make_kv(400, 1, 1, 128, T, torch.float16)
    x[0, 1, 0] = _codes_as_values(codes)
    check_contiguous(ref, x, 4, 8, 32, 32, codec=1)
