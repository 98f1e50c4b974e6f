"""RoPE over the launch shapes of swan_rope: rows with a wave of their own, and several
heads per wave; every row the same, bit for bit, as from a call of its own."""
import numpy as np
import pytest

import swan_inputs as si
from oracle import swan_oracle as O
from tests import swan_cases as C

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["f16", "f32"])
@pytest.mark.parametrize("batch,heads,n", [
    (1, 1, 1), (3, 5, 1), (1, 64, 64),             # a wave per row, up to 4096 rows
    (1, 3, 1400), (2, 7, 300), (1, 1, 5000),       # two heads at a time, odd head counts
    (5, 33, 90),
])
def test_rope_waves(gpu_device, swan_mod, torch_mod, dtype, batch, heads, n):
    """Every row of every launch shape, bit for bit the same as row by row."""
    torch = torch_mod
    pos0 = [1000 * b + 3 for b in range(batch)]
    x = torch.randn(batch, heads, n, 128, device=gpu_device,
                    generator=torch.Generator(gpu_device).manual_seed(n)).to(C.torch_dtype(dtype))
    y = swan_mod.rope(x, pos0, 10000.0)
    for b in range(batch):
        for h in {0, heads // 2, heads - 1}:
            for i in {0, n // 3, n - 1}:
                one = x[b, h, i].reshape(1, 1, 1, 128).contiguous()
                assert torch.equal(swan_mod.rope(one, [pos0[b] + i], 10000.0)[0, 0, 0], y[b, h, i])
    want = O.rope(x[0, heads - 1].cpu().numpy(), np.arange(pos0[0], pos0[0] + n), 10000.0,
                  si.np_dtype(dtype))
    got = y[0, heads - 1].cpu().numpy()
    if dtype == "f16":
        assert np.array_equal(got, want)
    else:  # one unit in the last place: float64 pow and sincos of two libraries
        assert np.all(np.abs(got - want) <= np.spacing(np.abs(want)))
