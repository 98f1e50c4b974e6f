"""Rotations of several problems in one call: each the same as from a call of its own
(bit for bit), at the edges of the row chunks, few rows (rank below 128), a matrix of
zeros, repeated singular values and scales near the ends of float32."""
import numpy as np
import pytest

import swan_inputs as si
from oracle import swan_oracle as O

pytestmark = pytest.mark.gpu


def _problems(torch, device):
    rng = si.rng_for(31)
    R = si.haar_orthogonal(rng, 128)
    S = [si.lowrank_rows(rng, n, R) for n in (1, 15, 16, 17, 127, 128, 512, 513, 4099)]
    S.append(np.zeros((40, 128)))
    S.append(np.concatenate([np.eye(128)] * 3))             # all singular values equal
    S.append(si.lowrank_rows(rng, 300, R) * 2.0 ** -60)
    S.append(si.lowrank_rows(rng, 300, R) * 2.0 ** 60)
    S += [rng.standard_normal((200, 128)) for _ in range(66 - len(S))]  # more than one launch
    return [torch.tensor(np.ascontiguousarray(x, dtype=np.float32), device=device) for x in S]


def test_batch_equals_single_calls(gpu_device, swan_mod, torch_mod):
    torch = torch_mod
    S = _problems(torch, gpu_device)
    P = torch.empty((len(S), 128, 128), device=gpu_device)
    sig = torch.empty((len(S), 128), device=gpu_device)
    swan_mod.calibrate_rotations(torch.cat(S), [x.shape[0] for x in S], P, sig)
    for i, x in enumerate(S):
        p1, s1 = torch.empty_like(P[i]), torch.empty_like(sig[i])
        swan_mod.calibrate_rotation(x, p1, s1)
        assert torch.equal(p1, P[i]) and torch.equal(s1, sig[i]), i
        # orthogonal, and the singular values of x in descending order
        p = p1.double().cpu().numpy()
        assert np.max(np.abs(p.T @ p - np.eye(128))) < 1e-6
        ref = O.calibrate(x.cpu().numpy())[1] if x.shape[0] >= 128 else None
        got = s1.double().cpu().numpy()
        assert np.all(np.diff(got) <= 0)
        if ref is not None:
            # float64 solve: 1e-15 of the largest eigenvalue, in sigma^2
            assert np.max(np.abs(got - ref)) <= 1e-6 * ref[0] + 1e-30


@pytest.mark.parametrize("flat", [True, False])
def test_channels_of_other_scales(gpu_device, swan_mod, torch_mod, flat):
    """Columns of S that differ in scale (outlier and nearly dead channels): the basis
    and each singular value to the float32 they are written in, also among the small
    channels, in one call with a problem whose columns have one scale."""
    torch = torch_mod
    rng = np.random.default_rng(11)
    scales, S = (1.0, 0.2, 1e-2, 1e-4, 1e-5, 1e-6, 1e-7), []
    for s in scales:
        x = rng.standard_normal((512, 128))
        if not flat:  # a falling spectrum in a rotated basis
            x = (x * np.exp(-np.arange(128) / 16)) @ si.haar_orthogonal(rng, 128)
        x[:, rng.permutation(128)[:16]] *= s
        if s == 1e-4:
            x[:, :2] *= 50.0
        S.append(x.astype(np.float32))
    P = torch.empty((len(S), 128, 128), device=gpu_device)
    sig = torch.empty((len(S), 128), device=gpu_device)
    swan_mod.calibrate_rotations(torch.tensor(np.concatenate(S), device=gpu_device),
                                 [512] * len(S), P, sig)
    for i, s in enumerate(scales):
        Po, so = O.calibrate(S[i])
        got = P[i].double().cpu().numpy()
        # signs by the oracle's column (its largest entry may tie to rounding)
        err = np.sqrt(np.sum((got * np.sign(np.sum(got * Po, axis=0)) - Po) ** 2, axis=0))
        # float32 P: 2^-24 of a unit column, doubled; the oracle's own float64 SVD:
        # 2^-53 of the largest singular value against the distance to the next one
        # (its square root of eigenvalues costs the rotated spectrum's 1 / 3000
        # smallest values another 1e-8 here)
        d = np.abs(np.diff(so))
        gap = np.minimum(np.r_[np.inf, d], np.r_[d, np.inf])
        tol = 2.0 ** -23 + 2.0 ** -53 * so[0] / gap + (0 if flat else 3e-8)
        assert np.all(err <= tol), (s, np.max(err / tol), np.max(err))
        rel = np.abs(sig[i].double().cpu().numpy() - so) / so
        assert np.all(rel <= 2.0 ** -23 + 2.0 ** -50 * so[0] / so), (s, np.max(rel))


def test_joint_outputs(gpu_device, torch_mod):
    """calibrate_joint into arrays of more heads than the layer's, into lists of matrices
    and on a stream of the caller's: the same matrices, in place on return; an output of
    another type is refused."""
    from paper_2511_18936_amd.layer import calibrate_joint

    torch = torch_mod
    Hq, Hkv, n, hidden = 4, 2, 70, 96
    gen = torch.Generator(device=gpu_device).manual_seed(5)
    rnd = lambda *s: torch.randn(s, device=gpu_device, generator=gen)
    args = (rnd(Hq, n, 128), rnd(Hkv, n, 128), rnd(Hkv, n, 128), rnd(Hq * 128, hidden), Hkv)
    ref = [torch.empty((Hkv, 128, 128), device=gpu_device) for _ in range(2)]
    calibrate_joint(*args, *ref)

    large = [torch.full((Hkv + 1, 128, 128), 7.0, device=gpu_device) for _ in range(2)]
    calibrate_joint(*args, *large)
    lists = [[torch.empty((128, 128), device=gpu_device) for _ in range(Hkv)] for _ in range(2)]
    calibrate_joint(*args, *lists)
    side = torch.cuda.Stream()
    other = [torch.zeros((Hkv, 128, 128), device=gpu_device) for _ in range(2)]
    torch.cuda.synchronize()
    calibrate_joint(*args, *other, stream=side)
    with torch.cuda.stream(torch.cuda.Stream()):  # waits for neither stream
        seen = [t.cpu() for t in other]
    for i in range(2):
        assert torch.equal(large[i][:Hkv], ref[i]) and torch.all(large[i][Hkv] == 7.0)
        assert torch.equal(torch.stack(lists[i]), ref[i])
        assert torch.equal(seen[i], ref[i].cpu())
    with pytest.raises(ValueError):
        calibrate_joint(*args, ref[0].half(), ref[1])


def _joint_args(torch, device, Hq=4, Hkv=2, n=70, hidden=96):
    gen = torch.Generator(device=device).manual_seed(5)
    rnd = lambda *s: torch.randn(s, device=device, generator=gen)
    return [rnd(Hq, n, 128), rnd(Hkv, n, 128), rnd(Hkv, n, 128), rnd(Hq * 128, hidden), Hkv]


def _joint_outputs(torch, device, Hkv=2):
    return [torch.zeros((Hkv, 128, 128), device=device) for _ in range(2)]


def test_joint_of_parameters(gpu_device, torch_mod):
    """W_o and the outputs may be a model's parameters, or made under inference mode."""
    from paper_2511_18936_amd.layer import calibrate_joint

    torch = torch_mod
    args, ref = _joint_args(torch, gpu_device), _joint_outputs(torch, gpu_device)
    calibrate_joint(*args, *ref)
    args[3] = torch.nn.Parameter(args[3])
    params = [torch.nn.Parameter(t) for t in _joint_outputs(torch, gpu_device)]
    calibrate_joint(*args, *params)
    lists = [[torch.nn.Parameter(m.clone()) for m in t] for t in _joint_outputs(torch, gpu_device)]
    calibrate_joint(*args, *lists)
    with torch.inference_mode():
        inf = _joint_outputs(torch, gpu_device)
    calibrate_joint(*args, *inf)
    for i in range(2):
        assert params[i].requires_grad and params[i].is_leaf
        assert torch.equal(params[i].detach(), ref[i])
        assert torch.equal(torch.stack([m.detach() for m in lists[i]]), ref[i])
        assert torch.equal(inf[i], ref[i])


def test_joint_refusals(gpu_device, swan_mod, torch_mod):
    """An output of another shape or layout, or an input on another device, is refused
    before anything is enqueued."""
    from paper_2511_18936_amd.layer import calibrate_joint

    torch = torch_mod
    args, ref = _joint_args(torch, gpu_device), _joint_outputs(torch, gpu_device)
    flat = torch.zeros((2, 128 * 128), device=gpu_device)
    wide = torch.zeros((2, 128, 256), device=gpu_device)[:, :, ::2]
    turned = torch.zeros((2, 128, 128), device=gpu_device).transpose(1, 2)
    for bad in (flat, wide, turned, [turned[0], ref[0][1]]):
        for out in ((bad, ref[1]), (ref[0], bad)):
            with pytest.raises(swan_mod.SwanError):
                calibrate_joint(*args, *out)
    for i in range(4):
        moved = list(args)
        moved[i] = args[i].cpu()
        with pytest.raises((ValueError, swan_mod.SwanError)):
            calibrate_joint(*moved, *ref)
    assert not any(t.any() for t in ref + [flat, wide, turned])


def test_joint_inputs_of_the_given_stream(gpu_device, torch_mod):
    """Inputs still being written on the caller's stream are read after that."""
    from paper_2511_18936_amd.layer import calibrate_joint

    torch = torch_mod
    args, ref = _joint_args(torch, gpu_device), _joint_outputs(torch, gpu_device)
    calibrate_joint(*args, *ref)
    late = [torch.zeros_like(t) for t in args[:4]]
    got = _joint_outputs(torch, gpu_device)
    big = torch.randn((4096, 4096), device=gpu_device)
    side = torch.cuda.Stream()
    torch.cuda.synchronize()
    with torch.cuda.stream(side):
        for _ in range(100):  # some milliseconds before the inputs are there
            big = (big @ big).clamp_(-1, 1)
        for dst, src in zip(late, args):
            dst.copy_(src)
    calibrate_joint(*late, args[4], *got, stream=side)
    torch.cuda.synchronize()
    for i in range(2):
        assert torch.equal(got[i], ref[i])


@pytest.mark.parametrize("budget", [1, 16 << 20, 40 << 20])
def test_joint_memory(gpu_device, torch_mod, monkeypatch, budget):
    """The joint matrices of many tokens are stacked and solved a group at a time, with the
    same result."""
    from paper_2511_18936_amd import layer, swan

    torch = torch_mod
    args = _joint_args(torch, gpu_device, Hq=6, Hkv=3, n=4096)
    ref, got = _joint_outputs(torch, gpu_device, 3), _joint_outputs(torch, gpu_device, 3)
    layer.calibrate_joint(*args, *ref)
    monkeypatch.setattr(layer, "JOINT_BYTES", budget, raising=False)
    torch.cuda.synchronize()
    torch.cuda.reset_peak_memory_stats()
    before = torch.cuda.memory_allocated()
    layer.calibrate_joint(*args, *got)
    peak = torch.cuda.max_memory_allocated() - before
    for i in range(2):
        assert torch.equal(got[i], ref[i])
    one = 3 * 4096 * 128 * 4 + swan.calibrate_workspace_bytes(128)  # an S_QK and its solver
    assert peak <= max(budget, one) + (1 << 20), peak  # and the rotations
