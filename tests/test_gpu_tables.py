"""Code tables built by workgroups of the encoder's own launch (run with -m gpu): payloads byte for byte against the oracle where
those workgroups have chunks of their own and where they do not, for all workgroup sizes, and which of the two a call takes."""
import pytest
import torch

from paper_2605_13734_amd import kvgen
from test_gpu_parity import check_contiguous
from test_gpu_routes import call_of, launches

pytestmark = pytest.mark.gpu


_DELTA = dict(bits_k=4, bits_v=4, transform=2, anchor_period=32)


def encoder_grid(**kw):
    """workgroups of the first encoder launch"""
    found = launches(call_of("compress", codec=1, **kw))
    return [grid for name, grid, _ in found if "encode_kernel" in name][0]


# chunks of 128 rows of K and V of 8 heads in workgroups of 8, 4 or 2; 22 workgroups build the tables
@pytest.mark.parametrize("T,kw,grid", [
    (128, dict(bits_k=4, bits_v=4), 4 + 22), (30000, dict(bits_k=4, bits_v=4), 470 + 22),
    (31360, dict(bits_k=4, bits_v=4), 490 + 22), (31361, dict(bits_k=4, bits_v=4), 492), (32768, dict(bits_k=4, bits_v=4), 512),
    (32769, dict(bits_k=4, bits_v=4), 1028 + 22), (16384, dict(bits_k=8, bits_v=8), 1024), (16385, dict(bits_k=8, bits_v=8), 1032 + 22),
    (16384, dict(bits_k=4, bits_v=4, group_k=128, group_v=128), 512), (15616, dict(bits_k=4, bits_v=4, group_k=128, group_v=128), 488 + 22),
    (24576, dict(bits_k=2, bits_v=2, group_k=64, group_v=64), 768), (24577, dict(bits_k=2, bits_v=2, group_k=64, group_v=64), 772 + 22),
    (65536, dict(bits_k=4, bits_v=2), 1024), (65537, dict(bits_k=4, bits_v=2), 1026 + 22),
    # kernels with the transforms take more registers: delta at groups of 64 two waves per SIMD (bf16 dense three), at 128 one, the rotation two
    (31360, dict(_DELTA, group_k=64), 490 + 22), (31361, dict(_DELTA, group_k=64), 492), (32768, dict(_DELTA, group_k=64), 512),
    (32769, dict(_DELTA, group_k=64), 514 + 22), (32769, dict(_DELTA, group_k=64, dtype=torch.bfloat16), 514 + 22),
    (49152, dict(_DELTA, group_k=64, dtype=torch.bfloat16), 768), (32768, dict(_DELTA, group_k=64, dtype=torch.bfloat16, paged=True), 512),
    (14976, dict(_DELTA, group_k=128), 234 + 22), (16384, dict(_DELTA, group_k=128), 256), (16385, dict(_DELTA, group_k=128), 258 + 22),
    (32768, dict(bits_k=4, bits_v=4, transform=1, group_k=128, dtype=torch.bfloat16, paged=True), 512)])
def test_who_builds(T, kw, grid):
    assert encoder_grid(L=1, H=8, T=T, **kw) == grid


@pytest.mark.parametrize("dtype,bits,group,T,peaked", [
    (torch.float16, 4, 32, 32768, False), (torch.float16, 4, 32, 32768, True),             # 512 threads, with chunks
    (torch.bfloat16, 8, 32, 16384, False), (torch.float16, 8, 32, 16300, True),            # 128
    (torch.float16, 3, 128, 16384, True),                                                  # 256
    (torch.float16, 2, 32, 32769, True), (torch.bfloat16, 4, 64, 200, True), (torch.float16, 8, 128, 130, True)])      # without
def test_tables_against_the_oracle(ref, dtype, bits, group, T, peaked):
    """peaked: nearly all codes of a tensor alike, in most of these cases so that tables exceed the length limit."""
    x = kvgen.make_kv(17, 1, 8, 128, T, dtype)
    if peaked:
        x = torch.where(torch.rand(x.shape, generator=torch.Generator().manual_seed(3)) < 0.03, x, x.abs() * 2.0 ** -9)
    check_contiguous(ref, x, bits, bits, group, group, codec=1)
