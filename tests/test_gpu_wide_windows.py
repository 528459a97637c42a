"""Windows of up to 32 requests that share the coder's launches, from 2^21 rows per tensor on (run with -m gpu): byte for byte
against calls of one request, and the launches on both sides of the lines."""
import numpy as np
import pytest
import torch

from paper_2605_13734_amd import kvc, kvgen
from test_gpu_parity import gpu_compress
from test_gpu_routes import call_of, encoders, launches

pytestmark = pytest.mark.gpu

_MIXED = dict(bits_k=0, bits_v=0, head_bits_k=[8, 2, 3, 8] * 128, head_bits_v=[2, 8, 2, 4] * 128)


@pytest.mark.parametrize("kw,dtype,paged", [
    (dict(bits_k=4, bits_v=4), torch.float16, False), (dict(bits_k=4, bits_v=4), torch.float16, True),
    (dict(bits_k=3, bits_v=2, group_v=64), torch.bfloat16, True), (dict(bits_k=8, bits_v=8, group_k=64, group_v=64), torch.bfloat16, False),
    (dict(bits_k=4, bits_v=4, transform=1), torch.float16, False),
    (dict(bits_k=2, bits_v=2, transform=2, anchor_period=16), torch.float16, True), (_MIXED, torch.float16, False)])
@pytest.mark.parametrize("n", [13, 33])
def test_wide_windows(n, kw, dtype, paged):
    """Ragged requests, an empty one in front and one inside; one request behind a full window of 32, or a window shared by K and V."""
    L, H, s = 64, 8, torch.cuda.current_stream().cuda_stream
    lens = [int(v) for v in torch.randint(1, 2 * (1 << 21) // (n * 500), (n,), generator=torch.Generator().manual_seed(n))]
    lens[0] = lens[9] = 0
    lens[5] += max(0, (1 << 21) // (L * H) + 1 - sum(lens))
    plan = kvc.Plan(kvc.F16 if dtype == torch.float16 else kvc.BF16, L, H, 128, codec=kvc.CODEC_HUFF8, max_tokens=max(lens), max_batch=n,
                    **dict(dict(group_k=32, group_v=32), **kw))
    src, dst, keep = [], [], []
    for i, t in enumerate(lens):
        if paged and t:
            pool, table = kvgen.make_paged(60 + i, L, H, 128, t, dtype, "cuda", 16)
            out = torch.zeros_like(pool)
            src.append(kvc.paged_request(pool, table, t))
            dst.append(kvc.paged_request(out, table, t))
        else:
            pool = kvgen.make_kv(60 + i, L, H, 128, t, dtype, "cuda") if t else torch.empty((L, 2, H, 0, 128), dtype=dtype, device="cuda")
            out, table = torch.zeros_like(pool), None
            src.append(kvc.contiguous_request(pool))
            dst.append(kvc.contiguous_request(out))
        keep.append((pool, table, out))
    buf = gpu_compress(plan, src, lens)
    buf.decompress(dst, s)
    torch.cuda.synchronize()
    assert not buf.status.any()
    for i in range(n):
        one = gpu_compress(plan, [src[i]], [lens[i]])
        assert np.array_equal(buf.payload_of(i), one.payload_of(0)), i
        got = keep[i][2].clone()
        keep[i][2].zero_()
        one.decompress([dst[i]], s)
        torch.cuda.synchronize()
        assert torch.equal(got.view(torch.int16), keep[i][2].view(torch.int16)), i


@pytest.mark.parametrize("n,T,kw,enc,dec", [
    (16, 1920, {}, [0, 1, 0, 1], 4), (16, 2048, {}, [2], 1), (17, 2048, {}, [0, 1], 2), (32, 1024, {}, [0, 1], 2), (33, 1024, {}, [0, 1, 2], 3),
    (4, 8192, {}, [2], 1), (5, 8192, {}, [2], 1), (5, 6528, {}, [0, 1], 2),
    (16, 6144, dict(group_k=64, group_v=64), [2], 1), (16, 6145, dict(group_k=64, group_v=64), [0, 1], 1)])
def test_lines_of_wide_windows(n, T, kw, enc, dec):
    """64 heads, rows counted in whole chunks of 128: 2^21 rows per tensor are 16 requests of 2048 tokens; groups of 64 share a launch up to 3 * 2^21 rows."""
    kw = dict(dict(bits_k=4, bits_v=4, group_k=32, group_v=32, codec=1), **kw)
    assert [kv for kv, _ in encoders(launches(call_of("compress", 8, 8, T, n=n, **kw)))] == enc
    assert sum("decode_kernel" in name for name, _, _ in launches(call_of("decompress", 8, 8, T, n=n, **kw))) == dec
