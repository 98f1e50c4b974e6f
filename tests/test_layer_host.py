"""The attention layer's call path on the host: what a prompt is projected by."""
import pytest

pytest.importorskip("paper_2511_18936_amd.swan")

from paper_2511_18936_amd.layer import SwanAttentionLayer  # noqa: E402


class _Cache:
    def append(self, *args):
        self.got = args


def _rows(x):
    return ("q", x), ("k", x), ("v", x)


@pytest.mark.parametrize("where", ["subclass", "object", "class"])
def test_a_prompt_goes_through_an_own_project(where, monkeypatch):
    """project() may be replaced (biases, normalised keys): a prompt's rows are its rows."""
    import torch

    class Own(SwanAttentionLayer):
        def project(self, x):
            return _rows(x)

    layer = (Own if where == "subclass" else SwanAttentionLayer).__new__(
        Own if where == "subclass" else SwanAttentionLayer)
    if where == "object":
        layer.project = _rows
    if where == "class":
        monkeypatch.setattr(SwanAttentionLayer, "project", lambda self, x: _rows(x))
    layer.n_heads = layer.n_kv_heads = 1
    layer.W_qkv = torch.zeros(4, 3 * 128)
    layer.P_qk, layer.cache = "P_qk", _Cache()
    x = torch.zeros(2, 5, 4)
    assert layer(x) is None
    assert layer.cache.got == (("k", x), ("v", x), "P_qk", None)
