"""Code tables built by workgroups of the encoder's own launch (run with -m gpu): payloads byte for byte against the oracle where
those workgroups have chunks of their own and where they do not, for all workgroup sizes, and which of the two a call takes."""
import heapq

import numpy as np
import pytest
import torch

from paper_2605_13734_amd import kvc, kvgen
from test_gpu_headbits import run
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


def longest_code(weights):
    """Length of the longest code of Huffman's algorithm without a limit (ties by symbol, then by age)."""
    queue, above, made = [(int(w), i) for i, w in enumerate(weights)], {}, 256
    heapq.heapify(queue)
    while len(queue) > 1:
        (a, i), (b, j) = heapq.heappop(queue), heapq.heappop(queue)
        above[i] = above[j] = made
        heapq.heappush(queue, (a + b, made))
        made += 1
    longest = 0
    for i in range(256):
        n = 0
        while i in above:
            i, n = above[i], n + 1
        longest = max(longest, n)
    return longest


def halvings(ref, x, bits_k, bits_v, group):
    """How often the weights of K's and V's table are halved, from the sample chunks of the packed codes."""
    L, _, H, T, _ = x.shape
    xu = kvgen.as_u16(x)
    cfg = ref.config(dtype=1, layers=L, heads=H, bits_k=bits_k, bits_v=bits_v, group_k=group, group_v=group)
    payload = ref.compress(cfg, xu[0, 0], xu[0, 1], ref.contiguous_layout(H, T, 128), T)
    sec, cph, out = kvc.payload_inspect(payload)[5], -(-T // 128), []
    for at, bits in ((6, bits_k), (8, bits_v)):
        codes = payload[sec[at]:sec[at] + sec[at + 1]].reshape(L * H, T, 16 * bits)
        count = np.zeros(256, dtype=np.int64)
        for c in {i * L * H * cph // 16 for i in range(16)}:
            count += np.bincount(codes[c // cph, c % cph * 128:c % cph * 128 + 128].ravel(), minlength=256)
        k = 0
        while longest_code((np.minimum(count, 1 << 18) + (1 << k)) >> k) > 12:
            k += 1
        out.append(k)
    return out


# (K and V in a launch, with chunks; without; a launch each, with chunks)
@pytest.mark.parametrize("bits_k,bits_v,group,T,share,grid", [
    (8, 8, 32, 16300, 0.03, 1024), (3, 3, 128, 16384, 0.01, 512), (2, 2, 32, 32769, 0.01, 1028 + 22),
    (4, 2, 128, 32768, 0.01, 512), (8, 4, 32, 32768, 0.03, 1024)])
def test_halved_tables(ref, bits_k, bits_v, group, T, share, grid):
    """Values that are zero but for a few: the first candidates of both tables exceed the length limit."""
    x = kvgen.make_kv(17, 1, 8, 128, T, torch.float16)
    x = torch.where(torch.rand(x.shape, generator=torch.Generator().manual_seed(3)) < share, x, torch.zeros(1, dtype=torch.float16))
    assert min(halvings(ref, x, bits_k, bits_v, group)) > 0
    assert encoder_grid(L=1, H=8, T=T, bits_k=bits_k, bits_v=bits_v, group_k=group, group_v=group) == grid
    check_contiguous(ref, x, bits_k, bits_v, group, group, codec=1)


@pytest.mark.parametrize("bits_k,bits_v,group,T,grid", [(4, 2, 128, 32768, 512), (8, 4, 32, 32768, 1024)])
def test_builders_with_chunks_in_a_launch_of_k(ref, bits_k, bits_v, group, T, grid):
    assert encoder_grid(L=1, H=8, T=T, bits_k=bits_k, bits_v=bits_v, group_k=group, group_v=group) == grid
    check_contiguous(ref, kvgen.make_kv(18, 1, 8, 128, T, torch.float16), bits_k, bits_v, group, group, codec=1)


def test_builders_with_chunks_and_width_tables(ref):
    """66 workgroups of the launch for K's eight heads of 2 bits build the tables of six launches."""
    tk, tv = [2] * 4 + [3] + [2] * 4 + [8], [4, 2, 8, 4, 2, 4, 4, 8, 2, 4]
    kw = dict(group_k=128, group_v=128, bits_k=0, bits_v=0, head_bits_k=tk, head_bits_v=tv)
    assert encoder_grid(L=1, H=10, T=32768, **kw) == 512
    run(ref, kvgen.make_kv(19, 1, 10, 128, 32768, torch.float16), np.array(tk, np.uint8), np.array(tv, np.uint8), 128, 128, codec=1)
