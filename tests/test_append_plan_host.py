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
    # different lengths: by the mean, or by a long one
    assert k(8, 0, [0] * 64, 200, [200, 40] * 32) == INSERT
    assert k(8, 0, [0] * 64, 400, [400, 50] * 32) == long
    assert k(8, 0, [0] * 64, 1000, ([1000] + [20] * 7) * 8) == long


@pytest.mark.parametrize("first,buffer", [(0, 0), (0, 33), (37, 16), (64, 128), (37, 0)])
def test_lengths_of_the_prefill_tests(first, buffer):
    """The batch that the prefill kernel's bit-exact tests append goes to that kernel."""
    per = [(0, 1, 31, 32, 33, 64, 95, 256, 257, 288, 299, 300)[i % 12] for i in range(64)]
    per = [300] + [max(n, 1 - first) if first == 0 else n for n in per[1:]]
    for dtype in (F16, E4M3):
        assert append_kernel(dtype, 2, buffer, [first] * 64, 300, per) == PREFILL
    assert append_kernel(F16, 2, 0, [0] * 64, 260) == PREFILL


@pytest.mark.parametrize("dtype,fresh,evicting,pruned", [
    # units from which 2, 4 and 8 tokens of each go to the kernel for few tokens
    (F16, (1200, 1400, 1800), (1200, 1400, 1800), (700, 900, 1300)),
    (F32, (1000, 1000, 1000), (860, 1120, 1640), (420, 540, 780)),
])
def test_few_tokens_of_many_units(dtype, fresh, evicting, pruned):
    for i, n in enumerate((2, 4, 8)):
        for buffer, cached, at in ((64, 0, fresh[i]), (64, 1000, evicting[i]), (0, 960, pruned[i])):
            heads = -(-at // 128)
            for h in (heads - 1, heads):
                want = FEW if 128 * h >= at else INSERT
                assert append_kernel(dtype, h, buffer, [cached] * 64, n) == want, (n, buffer, h)
    # more than 8: only where tokens are pruned, in blocks of 64 positions
    assert append_kernel(dtype, 32, 64, [0] * 64, 9) == INSERT
    assert append_kernel(dtype, 32, 0, [960] * 64, 16) == FEW
    assert append_kernel(dtype, 32, 0, [960] * 64, 17) == INSERT
    assert append_kernel(dtype, 32, 0, [1000] * 64, 32) == FEW  # over two pages
    assert append_kernel(dtype, 32, 0, [1000] * 64, 33) == INSERT
    # few sequences that append: as many blocks as those have
    assert append_kernel(dtype, 32, 64, [0] * 64, 4, [4] * 4 + [0] * 60) == INSERT
