"""Which launches a call consists of (run with -m gpu): the kernels, their dynamic LDS and their number on both sides of
the lines that the launch rules draw.  The call is captured, the nodes of the graph are read, nothing runs."""
import ctypes as C
import re

import pytest
import torch

from paper_2605_13734_amd import kvc, kvgen

pytestmark = pytest.mark.gpu


class _Dim3(C.Structure):
    _fields_ = [("x", C.c_uint), ("y", C.c_uint), ("z", C.c_uint)]


class _KernelNode(C.Structure):
    _fields_ = [("block", _Dim3), ("extra", C.c_void_p), ("func", C.c_void_p), ("grid", _Dim3), ("params", C.c_void_p),
                ("lds", C.c_uint)]


def _hip():
    with open("/proc/self/maps") as f:
        path = next(l.split()[-1] for l in f if "libamdhip64" in l)
    lib = C.CDLL(path)
    lib.hipKernelNameRefByPtr.restype = C.c_char_p
    lib.hipKernelNameRefByPtr.argtypes = [C.c_void_p, C.c_void_p]
    return lib


def launches(call):
    """[(kernel, workgroups, dynamic LDS)] of what `call(stream)` enqueues."""
    hip, g, side = _hip(), torch.cuda.CUDAGraph(keep_graph=True), torch.cuda.Stream()
    with torch.cuda.graph(g, stream=side):
        call(side.cuda_stream)
    n, graph = C.c_size_t(0), C.c_void_p(g.raw_cuda_graph())
    assert hip.hipGraphGetNodes(graph, None, C.byref(n)) == 0
    nodes = (C.c_void_p * n.value)()
    assert hip.hipGraphGetNodes(graph, nodes, C.byref(n)) == 0
    out = []
    for node in nodes:
        p = _KernelNode()
        assert hip.hipGraphKernelNodeGetParams(C.c_void_p(node), C.byref(p)) == 0
        name = hip.hipKernelNameRefByPtr(p.func, None).decode()
        out.append((name, p.grid.x * p.grid.y, p.lds))
    return out


def call_of(direction, L, H, T, n=1, dtype=torch.float16, paged=False, **strategy):
    """A compress or decompress call over n requests of T tokens (one tensor for all: nothing runs)."""
    code = kvc.F16 if dtype == torch.float16 else kvc.BF16
    plan = kvc.Plan(code, L, H, 128, max_tokens=T, max_batch=n, **strategy)
    sizes = [plan.payload_size(T)[0]] * n
    offsets = [0]
    for s in sizes:
        offsets.append(offsets[-1] + (s + 255) // 256 * 256)
    if paged:
        pages = -(-T // 16)
        x = torch.empty((L, 2, pages, 16, H, 128), dtype=dtype, device="cuda")
        table = kvgen.block_table(3, pages, pages, "cuda")
        reqs = [kvc.paged_request(x, table, T)] * n
    else:
        table = None
        x = torch.empty((L, 2, H, T, 128), dtype=dtype, device="cuda")
        reqs = [kvc.contiguous_request(x)] * n
    payload = torch.empty(offsets[-1], dtype=torch.uint8, device="cuda")
    words = torch.zeros(2 * n, dtype=torch.int64, device="cuda")
    ws = torch.empty(max(plan.workspace_size(), 256), dtype=torch.uint8, device="cuda")

    def call(stream):
        if direction == "compress":
            kvc.compress(plan, reqs, payload.data_ptr(), offsets, words.data_ptr(), words[n:].data_ptr(), ws.data_ptr(), stream)
        else:
            kvc.decompress(plan, payload.data_ptr(), offsets, reqs, words[n:].data_ptr(), ws.data_ptr(), stream)
    call.keep = (x, table, payload, words, ws)
    return call


def lds_of(found, kernel):
    sizes = {lds for name, _, lds in found if kernel in name}
    assert len(sizes) == 1, (kernel, found)
    return sizes.pop()


@pytest.mark.parametrize("dtype", [torch.float16, torch.bfloat16])
@pytest.mark.parametrize("bits", [2, 3, 4, 8])
@pytest.mark.parametrize("paged", [False, True])
def test_bound_on_the_workgroups_of_a_unit(bits, paged, dtype):
    """Kernels that gain nothing from a smaller window of the tensor, or lose by it, run without the bound."""
    f16 = dtype == torch.float16
    L, H, T = 4, 8, 300                                  # (K and V groups differ: three launches at any size)
    kw = dict(dtype=dtype, paged=paged, bits_k=bits, bits_v=bits, group_v=64)
    wide = bits == 8 or (bits == 4 and f16)
    for group in (32, 128):
        found = launches(call_of("compress", L, H, T, group_k=group, **kw))
        assert len(found) == 3
        assert lds_of(found, "compress_k_kernel") == (32000 if paged and wide and group == 32 else 0)
        assert lds_of(found, "compress_v_kernel") == (32000 if paged and f16 else 0)
    found = launches(call_of("decompress", L, H, T, group_k=32, **kw))
    want = (40000 if bits == 4 else 0) if paged else (40000 if bits <= 4 else 0)
    assert lds_of(found, "decompress_k_kernel") == want and lds_of(found, "decompress_v_kernel") == want
    if paged:                                            # 2^19 rows and more
        found = launches(call_of("decompress", 8, 8, 8192, group_k=32, **kw))
        want = 40000 if bits in (4, 8) or (bits == 2 and not f16) else 0
        assert lds_of(found, "decompress_k_kernel") == want and lds_of(found, "decompress_v_kernel") == want


@pytest.mark.parametrize("T", [16384 - 128, 16384])
def test_bound_of_large_compressions(T):
    """2^20 rows: below, a tensor is a few generations of workgroups and has no window to keep small."""
    for bits, group, lds in ((4, 32, 40000), (3, 32, 36000), (3, 128, 40000)):
        found = launches(call_of("compress", 8, 8, T, bits_k=bits, bits_v=bits, group_k=group, group_v=64))
        assert lds_of(found, "compress_k_kernel") == (lds if T == 16384 else 0)
        assert lds_of(found, "compress_v_kernel") == 0


@pytest.mark.parametrize("T,lds", [(65536 - 32, 40000), (65536, 32000)])
def test_bound_of_large_four_bit_decompressions(T, lds):
    found = launches(call_of("decompress", 8, 8, T, bits_k=4, bits_v=4, group_k=32, group_v=64))
    assert lds_of(found, "decompress_k_kernel") == lds and lds_of(found, "decompress_v_kernel") == lds


@pytest.mark.parametrize("bits,lds", [(2, 40000), (3, 32000), (4, 32000), (8, 0)])
def test_bound_of_decompressions_of_many_requests(bits, lds):
    """Eight requests in a launch, just below 2^21 rows together and 2^21."""
    for T, want in ((4096 - 32, 40000 if bits < 8 else 0), (4096, lds)):
        found = launches(call_of("decompress", 8, 8, T, n=8, bits_k=bits, bits_v=bits, group_k=32, group_v=64))
        assert lds_of(found, "decompress_k_kernel") == want and lds_of(found, "decompress_v_kernel") == want


def decompress_shape(found, bits):
    """(dynamic LDS, waits between the stores) of the decompressions of one width, the same for K and V."""
    shapes = set()
    for name, _, lds in found:
        m = re.search(r"decompress_[kv]_kernelILi%dELi\dELb\dELi\dELb(\d)E" % bits, name)
        if m:
            shapes.add((lds, int(m.group(1))))
    assert len(shapes) == 1, found
    return shapes.pop()


_HALF, _BF = torch.float16, torch.bfloat16


@pytest.mark.parametrize("dtype,bits,group,lines", [
    (_HALF, 4, 32, [(8192, 40000, 1), (32736, 40000, 1), (32768, 52000, 1), (98272, 52000, 1), (98304, 52000, 0)]),
    (_HALF, 4, 128, [(32736, 40000, 1), (32768, 52000, 0), (98304, 52000, 0)]),
    (_BF, 4, 64, [(32768, 52000, 1), (98304, 52000, 0)]),
    (_HALF, 2, 64, [(10208, 52000, 1), (10240, 40000, 0), (14304, 40000, 0), (14336, 32000, 1), (98304, 40000, 0)]),
    (_HALF, 2, 32, [(10208, 52000, 1), (10240, 32000, 1), (98304, 32000, 1)]),
    (_BF, 2, 128, [(10240, 40000, 0), (14336, 40000, 1)]),
    (_BF, 2, 32, [(10240, 40000, 1)]),
    (_HALF, 3, 32, [(8160, 32000, 0), (8192, 40000, 0)]), (_BF, 3, 32, [(8160, 32000, 0), (8192, 40000, 1)]),
    (_BF, 8, 32, [(4096, 52000, 0), (8160, 52000, 0), (8192, 52000, 1)])])
def test_shapes_of_paged_decompressions(dtype, bits, group, lines):
    """Both sides of every line that the type, the group and the rows (256 heads of T tokens) draw."""
    for T, lds, paced in lines:
        found = launches(call_of("decompress", 32, 8, T, dtype=dtype, paged=True, bits_k=bits, bits_v=bits, group_k=group, group_v=group))
        assert decompress_shape(found, bits) == (lds, paced), T


@pytest.mark.parametrize("dtype,bits,group,lines", [
    (_HALF, 3, 64, [(10208, 80000), (10240, 40000), (98272, 40000), (98304, 80000)]),
    (_HALF, 3, 32, [(10240, 80000)]), (_BF, 3, 64, [(10240, 80000)]), (_BF, 3, 128, [(10240, 40000)]),
    (_HALF, 2, 64, [(24544, 80000), (24576, 40000), (98272, 40000), (98304, 80000)]),
    (_HALF, 2, 32, [(24576, 80000)]), (_BF, 2, 64, [(24576, 80000)]),
    (_HALF, 8, 32, [(8192, 80000)]), (_HALF, 4, 32, [(24544, 32000), (24576, 80000)])])
def test_shapes_of_dense_decompressions(dtype, bits, group, lines):
    for T, lds in lines:
        found = launches(call_of("decompress", 32, 8, T, dtype=dtype, bits_k=bits, bits_v=bits, group_k=group, group_v=group))
        assert decompress_shape(found, bits) == (lds, 0), T


@pytest.mark.parametrize("paged,dtype,bits,group,lines", [
    (False, _HALF, 2, 32, [(3040, 40000, 0), (3072, 80000, 0)]), (False, _HALF, 3, 64, [(3040, 32000, 0), (3072, 40000, 0)]),
    (False, _BF, 2, 64, [(3072, 40000, 0)]), (False, _HALF, 4, 64, [(6112, 32000, 0), (6144, 80000, 0)]),
    (True, _HALF, 2, 32, [(2528, 52000, 1), (2560, 40000, 0)]), (True, _BF, 2, 32, [(2560, 40000, 1)]),
    (True, _BF, 2, 64, [(2560, 40000, 0)]), (True, _HALF, 4, 32, [(8160, 40000, 1)])])
def test_shapes_of_decompressions_of_four_requests(paged, dtype, bits, group, lines):
    for T, lds, paced in lines:
        found = launches(call_of("decompress", 32, 8, T, n=4, dtype=dtype, paged=paged, bits_k=bits, bits_v=bits, group_k=group, group_v=group))
        assert decompress_shape(found, bits) == (lds, paced), T


def test_shapes_of_paged_decompressions_by_head():
    """Launches over some of the heads (width tables) have no waits below 5 * 2^19 rows."""
    tab = dict(head_bits_k=[8, 2] * 128, head_bits_v=[2, 8] * 128)
    for T, want in ((20448, ((40000, 0), (40000, 0))), (20480, ((52000, 1), (40000, 1)))):
        found = launches(call_of("decompress", 32, 8, T, dtype=_BF, paged=True, **tab))
        assert (decompress_shape(found, 8), decompress_shape(found, 2)) == want


def test_shapes_of_large_decompressions_with_a_transform():
    def lds(T, paged=False, **kw):
        found = launches(call_of("decompress", 32, 8, T, paged=paged, bits_v=kw["bits_k"], **kw))
        return lds_of(found, "decompress_k_kernel"), lds_of(found, "decompress_v_kernel")
    for paged, want in ((False, 32000), (True, 40000)):
        assert lds(98304, paged, bits_k=8, transform=1) == (want, want) and lds(98272, paged, bits_k=8, transform=1) == (0, 0)
        assert lds(98304, paged, bits_k=4, transform=1) == (0, 0)
    delta = dict(bits_k=4, transform=2, anchor_period=32)
    assert lds(16384, **delta) == (40000, 40000) and lds(16352, **delta) == (0, 0) and lds(16384, True, **delta) == (0, 0)
    assert lds(16384, bits_k=4, transform=2, anchor_period=16) == (0, 0)


@pytest.mark.parametrize("bits,lds", [(2, 24000), (4, 24000), (8, 32000)])
@pytest.mark.parametrize("group", [32, 64, 128])
def test_bound_of_paged_bf16_v_compressions(group, bits, lds):
    """V units are one pass of few registers whatever their group."""
    for T, want in ((6112, 0), (6144, lds)):
        found = launches(call_of("compress", 32, 8, T, dtype=_BF, paged=True, bits_k=bits, bits_v=bits, group_k=64, group_v=group))
        assert lds_of(found, "compress_v_kernel") == want and lds_of(found, "compress_k_kernel") == 0


def test_bound_of_one_launch_bf16_compressions():
    for dtype, group, T, want in ((_BF, 32, 4064, 0), (_BF, 32, 4096, 32000), (_BF, 64, 4096, 0), (_HALF, 32, 4096, 0)):
        found = launches(call_of("compress", 32, 8, T, dtype=dtype, bits_k=4, bits_v=4, group_k=group, group_v=group))
        assert len(found) == 1 and lds_of(found, "compress_call_kernel") == want


@pytest.mark.parametrize("kw", [dict(transform=1), dict(transform=2, anchor_period=16)])
def test_no_bound_with_a_transform(kw):
    for direction in ("compress", "decompress"):
        assert all(lds == 0 for _, _, lds in launches(call_of(direction, 2, 4, 200, group_k=64, group_v=32, **kw)))


@pytest.mark.parametrize("bits,group", [(2, 64), (4, 32), (8, 128)])
def test_one_launch_below_two_mebirows(bits, group):
    """Decompression in one launch reads and writes the same window of the tensor as in three."""
    for T, n in ((32768 - 32, 1), (32768, 3)):
        for direction in ("compress", "decompress"):
            found = launches(call_of(direction, 8, 8, T, bits_k=bits, bits_v=bits, group_k=group, group_v=group))
            assert len(found) == n
            if n == 1:
                assert lds_of(found, "_call_kernel") == (40000 if direction == "decompress" else 0)


def encoders(found):
    """(tensor: 0 K, 1 V, 2 both; chunks per workgroup) of the encoder launches."""
    names = [re.search(r"encode_kernelILi\d+ELi\d+ELi\dELi(\d)ELb\dELb\dELi(\d)E", name) for name, _, _ in found]
    return [(int(m.group(1)), int(m.group(2))) for m in names if m]


@pytest.mark.parametrize("dtype,paged,bits,group,L,T,shared", [
    (torch.bfloat16, True, 4, 128, 1, 8192, True), (torch.bfloat16, True, 4, 128, 1, 8193, False),      # one wave per SIMD
    (torch.bfloat16, True, 8, 128, 1, 8193, False), (torch.bfloat16, False, 4, 128, 1, 8193, True),
    (torch.float16, False, 4, 128, 8, 16384, True), (torch.float16, False, 4, 128, 8, 16385, False),    # two
    (torch.float16, True, 2, 128, 8, 16384, True), (torch.float16, False, 8, 128, 8, 16385, True),
    (torch.bfloat16, True, 4, 64, 8, 16385, True), (torch.float16, False, 4, 64, 8, 32768, False),
    (torch.float16, False, 4, 32, 8, 32768, True)])
def test_encoder_shares_a_launch_where_it_pays(dtype, paged, bits, group, L, T, shared):
    found = launches(call_of("compress", L, 8, T, dtype=dtype, paged=paged, bits_k=bits, bits_v=bits, group_k=group, group_v=group, codec=1))
    assert [kv for kv, _ in encoders(found)] == ([2] if shared else [0, 1])


@pytest.mark.parametrize("T,lds", [(6144, 0), (6145, 40000), (10240, 40000), (10241, 0)])
@pytest.mark.parametrize("dtype", [torch.float16, torch.bfloat16])
def test_bound_of_rotated_encoders(dtype, T, lds):
    """More than three and up to five workgroups per compute unit, 16 per 128 tokens: K blocks of 64 rows go two at a time."""
    def bounds(**kw):
        found = launches(call_of("compress", 8, 8, T, dtype=dtype, codec=1, transform=1, **kw))
        return [size for name, _, size in found if "encode_kernel" in name]
    assert bounds(bits_k=4, bits_v=4, group_k=64, group_v=64) == [lds, 0]
    assert bounds(bits_k=2, bits_v=3, group_k=64, group_v=32) == [lds, 0]
    for kw in (dict(bits_k=8, bits_v=8, group_k=64), dict(bits_k=4, bits_v=4, group_k=32), dict(bits_k=4, bits_v=4, group_k=128)):
        assert bounds(group_v=64, **kw) == [0, 0]


@pytest.mark.parametrize("n,want", [(1, [2]), (4, [2]), (5, [0, 1]), (8, [0, 1]), (11, [0, 1, 2])])
def test_encoder_windows(n, want):
    """Up to four requests share a launch for K and V, more of them take the passes apart, eight at a time."""
    found = launches(call_of("compress", 1, 4, 700, n=n, bits_k=4, bits_v=4, codec=1))
    assert [kv for kv, _ in encoders(found)] == want
    found = launches(call_of("compress", 1, 4, 700, n=n, bits_k=8, bits_v=8, codec=1))
    assert [kv for kv, _ in encoders(found)] == [2] * -(-n // 4)                  # (8 bits: four at a time)


@pytest.mark.parametrize("n,enc,dec", [(15, [0, 1, 0, 1], 2), (16, [0, 1, 0, 1], 2), (17, [0, 1, 0, 1], 2), (24, [0, 1, 0, 1], 2),
                                        (25, [0, 1, 0, 1, 2], 3), (36, [0, 1] * 3, 3)])
def test_coder_windows_of_many_requests(n, enc, dec):
    """Eight requests a window, from seventeen on twelve; a rest of up to four shares its launch for K and V."""
    found = launches(call_of("compress", 1, 4, 700, n=n, bits_k=4, bits_v=4, codec=1))
    assert [kv for kv, _ in encoders(found)] == enc
    for kw in (dict(bits_k=4, bits_v=2), dict(bits_k=4, bits_v=4, transform=1), dict(bits_k=4, bits_v=4, transform=2, anchor_period=16)):
        found = launches(call_of("decompress", 1, 4, 700, n=n, codec=1, **kw))
        assert sum("decode_kernel" in name for name, _, _ in found) == 2 * dec
        found = launches(call_of("compress", 1, 4, 700, n=n, codec=1, **kw))
        assert sum("encode_kernel" in name for name, _, _ in found) == 2 * dec


_MIXED = dict(head_bits_k=[8, 2] * 32, head_bits_v=[2, 8] * 32)


@pytest.mark.parametrize("kw,T,n,windows", [
    (dict(bits_k=8, bits_v=8, transform=1), 256, 24, 2), (dict(bits_k=8, bits_v=8, transform=1), 257, 24, 3),      # 1536 and 2304 of 2048
    (dict(bits_k=8, bits_v=8, transform=1), 385, 24, 2), (dict(bits_k=8, bits_v=8, transform=1), 257, 23, 2),      # 3072; a window less
    (dict(bits_k=4, bits_v=4, transform=1), 640, 24, 2), (dict(bits_k=4, bits_v=4, transform=1), 641, 24, 3),      # 3840 and 4608 of 4096
    (dict(bits_k=4, bits_v=4, transform=1), 769, 24, 2), (dict(bits_k=4, bits_v=8, transform=1), 257, 32, 4),      # 5376; V alone
    (dict(bits_k=4, bits_v=8, transform=1), 641, 32, 3),                                                           # (K is not the widest)
    (_MIXED, 640, 24, 2), (_MIXED, 641, 24, 3), (_MIXED, 1024, 24, 3), (_MIXED, 1025, 24, 2)])
def test_coder_windows_with_a_small_rest(kw, T, n, windows):
    """Requests of 64 heads: windows of twelve, but eight where the launches of twelve of the widest codes have up to a quarter more chunks
    than are resident (16 per compute unit, at 8 bits 8), with width tables up to a half."""
    found = launches(call_of("compress", 8, 8, T, n=n, codec=1, **kw))
    assert sum("encode_kernel" in name for name, _, _ in found) == (4 if "head_bits_k" in kw else 2) * windows
    if "transform" in kw:
        found = launches(call_of("decompress", 8, 8, T, n=n, codec=1, **kw))
        assert sum("decode_kernel" in name for name, _, _ in found) == 2 * windows


@pytest.mark.parametrize("n", [1, 4, 5, 8])
def test_decoder_windows(n):
    """Width tables: where K or V has a width of its own, more than four requests keep K and V apart."""
    def decoders(tab_k, tab_v):
        found = launches(call_of("decompress", 1, 4, 300, n=n, head_bits_k=tab_k, head_bits_v=tab_v, codec=1))
        return sum("decode_kernel" in name for name, _, _ in found)
    assert decoders([8, 2, 2, 8], [2, 8, 8, 8]) == (2 if n <= 4 else 4)
    assert decoders([4, 3, 3, 4], [4, 2, 4, 2]) == (3 if n <= 4 else 4)
    assert decoders([3, 3, 3, 3], [4, 2, 4, 2]) == 3


@pytest.mark.parametrize("paged,bits,group,n,lines", [
    (False, 3, 64, 1, [(2432, 0), (2560, 14000), (3072, 14000)]), (False, 3, 32, 1, [(2944, 0), (3072, 40000)]),
    (False, 2, 64, 1, [(2944, 0), (3072, 14000)]),
    (False, 4, 64, 1, [(32640, 0), (32768, 14000), (98304, 0)]), (False, 4, 32, 1, [(32768, 0)]),
    (False, 3, 32, 4, [(8064, 14000), (8192, 40000), (24576, 14000)]), (False, 2, 32, 4, [(8064, 0), (8192, 14000), (24576, 0)]),
    (False, 3, 64, 4, [(24448, 40000), (24576, 14000)]), (False, 3, 128, 4, [(24576, 40000)]),
    (True, 2, 64, 1, [(2432, 0), (2560, 14000), (32768, 14000), (98304, 0)]), (True, 2, 32, 1, [(2560, 14000), (32768, 0)]),
    (True, 3, 64, 1, [(32640, 14000), (32768, 0)]), (True, 3, 32, 4, [(8064, 0), (8192, 14000), (24576, 0)]),
    (True, 3, 32, 1, [(2432, 0), (2560, 40000), (10624, 40000), (10752, 14000), (32640, 14000), (32768, 0)]), (True, 4, 64, 1, [(8192, 0)])])
def test_shapes_of_decoders(paged, bits, group, n, lines):
    """Both sides of the lines: 256 heads of T tokens, or four requests of 64 heads, are T workgroups for K and V together, T / 2
    for one of them (from 2^23 rows on)."""
    for T, lds in lines:
        layers = 32 if n == 1 else 8
        found = launches(call_of("decompress", layers, 8, T, n=n, paged=paged, bits_k=bits, bits_v=bits, group_k=group, group_v=group, codec=1))
        assert lds_of(found, "decode_kernel") == lds, T


@pytest.mark.parametrize("n,T,waves", [
    (1, 8192, 4), (1, 8193, 8), (1, 16384, 8), (1, 16385, 4), (1, 20480, 4), (1, 20481, 8), (1, 32768, 8), (1, 32769, 4),
    (2, 8192, 8), (2, 8193, 4), (4, 4800, 4), (4, 6144, 4), (4, 6145, 8), (4, 8192, 8), (4, 8193, 4)])
def test_chunks_per_encoder_workgroup(n, T, waves):
    """16 chunks per 128 tokens, 256 compute units: eight per workgroup above 1024 chunks and up to 4096, but for 2049 to
    3072 chunks unless 2560 of them are one request's."""
    found = launches(call_of("compress", 1, 8, T, n=n, bits_k=4, bits_v=4, codec=1))
    assert encoders(found) == [(2, waves)]
