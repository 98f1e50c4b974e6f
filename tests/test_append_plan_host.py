"""Which kernel an append runs, from its lengths alone (host arithmetic): the rule looks at
the tokens of the sequences, never at the stride of the rows they come in."""
import ctypes

import pytest

swan = pytest.importorskip("paper_2511_18936_amd.swan")

NONE, STEP, INSERT, PREFILL, FEW = range(5)
F32, F16, E4M3 = swan.SWAN_F32, swan.SWAN_F16, swan.SWAN_F16_E4M3


def append_kernel(dtype, heads, buffer, lens, n_new, per=None):
    a = lambda v: None if v is None else (ctypes.c_int32 * len(v))(*v)
    return swan.lib().swan_append_kernel(dtype, len(lens), heads, buffer, a(lens), n_new, a(per))


@pytest.mark.parametrize("dtype", [F32, F16, E4M3])
def test_rule(dtype):
    long = INSERT if dtype == F32 else PREFILL
    k = lambda *a: append_kernel(dtype, *a)
    assert k(8, 64, [0] * 64, 1) == STEP and k(8, 64, [0] * 64, 0) == NONE
    assert k(8, 64, [5] * 64, 256, [0] * 64) == NONE
    # 1024 units: 64 tokens each, whatever the rows' stride; 160 and more
    assert k(8, 0, [0] * 64, 64) == INSERT
    assert k(8, 0, [0] * 64, 256, [64] * 64) == INSERT
    assert k(8, 0, [0] * 64, 4096, [64] * 64) == INSERT
    assert k(8, 0, [0] * 64, 159) == INSERT
    assert k(8, 0, [0] * 64, 160) == long
    assert k(8, 0, [1000] * 64, 4096, [160] * 64) == long
    # sequences that append nothing do not count
    assert k(8, 0, [0] * 64, 160, [160] * 32 + [0] * 32) == long
    # 512 blocks of 64 positions are too few
    assert k(8, 0, [0] * 16, 128) == INSERT
    assert k(8, 0, [0] * 8, 256) == INSERT
    assert k(8, 0, [0] * 8, 257) == long
    assert k(8, 0, [0], 1009) == INSERT
    # different lengths: by the mean, unless a few long ones make it
    assert k(8, 0, [0] * 64, 200, [200, 40] * 32) == INSERT
    assert k(8, 0, [0] * 64, 256, [256, 64] * 32) == long
    assert k(8, 0, [0] * 64, 400, [400, 100] * 32) == long
    assert k(8, 0, [0] * 64, 700, ([700] + [200] * 3) * 16) == long
    assert k(8, 0, [0] * 64, 4000, ([4000] + [100] * 7) * 8) == long
    assert k(8, 0, [0] * 64, 300, ([300] + [20] * 7) * 8) == INSERT
    assert k(8, 0, [0] * 64, 1000, ([1000] + [20] * 7) * 8) == INSERT
    assert k(8, 0, [0] * 64, 2000, ([2000] + [100] * 7) * 8) == INSERT


@pytest.mark.parametrize("first,buffer", [(0, 0), (0, 33), (37, 16), (64, 128), (37, 0)])
def test_lengths_of_the_prefill_tests(first, buffer):
    """The batch that the prefill kernel's bit-exact tests append goes to that kernel."""
    per = [(0, 1, 31, 32, 33, 64, 95, 256, 257, 288, 299, 300)[i % 12] for i in range(64)]
    per = [300] + [max(n, 1 - first) if first == 0 else n for n in per[1:]]
    for dtype in (F16, E4M3):
        assert append_kernel(dtype, 2, buffer, [first] * 64, 300, per) == PREFILL
    assert append_kernel(F16, 2, 0, [0] * 64, 260) == PREFILL


@pytest.mark.parametrize("dtype,buffer,cached,few,insert", [
    # (units, tokens of each) that the kernel for few tokens takes, or that go by
    (F16, 128, 0, [(2048, 2), (2048, 8), (4096, 8)], [(256, 2), (1024, 4), (2048, 16), (4096, 24)]),
    (F16, 64, 1000, [(2048, 4), (4096, 8)], [(768, 4), (1024, 8), (4096, 12)]),
    (F16, 0, 960, [(768, 2), (2048, 8), (4096, 20)], [(512, 8), (1152, 16), (4096, 32)]),
    (F16, 0, 1000, [(1024, 12), (4096, 16), (4096, 32)], [(512, 24), (2048, 48)]),
    (F32, 128, 0, [(2048, 4), (4096, 8)], [(640, 8), (1024, 16), (4096, 32)]),
    (F32, 64, 1000, [(2048, 2), (4096, 8)], [(640, 4), (1024, 12), (4096, 16)]),
    (F32, 0, 960, [(640, 3), (2048, 12), (4096, 20)], [(512, 8), (896, 16), (4096, 32)]),
    (F32, 0, 1000, [(1280, 16), (4096, 32)], [(512, 16), (4096, 64)]),
])
def test_few_tokens_of_many_units(dtype, buffer, cached, few, insert):
    """Sizes where one of the two kernels measured faster by a tenth or more."""
    for sizes, want in ((few, FEW), (insert, INSERT)):
        for units, n in sizes:
            got = append_kernel(dtype, units // 128, buffer, [cached] * 64, n)
            assert got == want, (units, n)


def test_few_tokens_of_some_sequences():
    """By the sequences that append, and what all of them append."""
    assert append_kernel(F16, 32, 64, [0] * 64, 4, [4] * 64) == FEW
    assert append_kernel(F16, 32, 64, [0] * 64, 4, [4] * 4 + [0] * 60) == INSERT
    assert append_kernel(F16, 32, 0, [1000] * 64, 300, [300] + [2] * 63) == FEW
    assert append_kernel(F16, 32, 0, [1000] * 64, 300, [300] + [60] * 63) == INSERT
