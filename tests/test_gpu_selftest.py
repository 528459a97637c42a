"""Device self-test (run with -m gpu): the instruction sequences the quantizer kernels use in
place of IEEE division and subtraction give the IEEE result on every input of their domain."""
import pytest
import torch

from paper_2605_13734_amd import kvc

pytestmark = pytest.mark.gpu

NAMES = ["range/3", "range/7", "range/15", "range/255", "1/scale", "x-zero (packed fp16)", "float->byte"]


def test_arithmetic_shortcuts_are_exact():
    counts = torch.full((kvc.SELFTEST_COUNTS,), -1, dtype=torch.int64, device="cuda:0")
    rc = kvc.selftest(counts.data_ptr(), torch.cuda.current_stream().cuda_stream)
    assert rc == 0
    torch.cuda.synchronize()
    got = counts.cpu().tolist()
    print("selftest mismatch counts:", dict(zip(NAMES, got)))
    assert got[:len(NAMES)] == [0] * len(NAMES), dict(zip(NAMES, got))
    assert got[len(NAMES):] == [0] * (kvc.SELFTEST_COUNTS - len(NAMES))


def test_place_scan_waits():
    """The encoder's scanner gives up on a running workgroup that reports nothing, not on one that other work on the GPU
    keeps from starting: the self-test lets the last of three start twenty times the scanner's limit late.  Where one of
    them never reports, the others stop within 50 ms, and nothing is placed or closed, by the next launch either; one
    that never starts is waited for as long as the scanner is told."""
    counts = torch.full((kvc.SELFTEST_COUNTS,), -1, dtype=torch.int64, device="cuda:0")
    assert kvc.selftest(counts.data_ptr(), torch.cuda.current_stream().cuda_stream) == 0
    torch.cuda.synchronize()
    assert counts.cpu().tolist()[7] == 0


def test_code_table_waits():
    """The encoder's wait for a code table (same count): found by all waves of a workgroup when its words come one after the other and
    the first candidate is too long; given up, with status and carry word marked, where no table or one word of it never comes."""
    counts = torch.full((kvc.SELFTEST_COUNTS,), -1, dtype=torch.int64, device="cuda:0")
    assert kvc.selftest(counts.data_ptr(), torch.cuda.current_stream().cuda_stream) == 0
    torch.cuda.synchronize()
    assert counts.cpu().tolist()[7] == 0
