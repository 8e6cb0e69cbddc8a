"""What BayesianLinear takes beside dense arrays on the current device, which the native calls leave to the general path: the same
results, the same refusals."""
import gc
import threading

import pytest
import torch

pytestmark = pytest.mark.gpu
DEV = "cuda"
K, O, S = 96, 130, 3


def _layer(rows, own, bias=True, seed=5):
    from paper_2604_04736_amd.autograd import BayesianLinear
    g = torch.Generator(device=DEV).manual_seed(rows)
    x = torch.randn(*((S, rows, K) if own else (rows, K)), device=DEV, generator=g)
    p = [torch.randn(O, K, device=DEV, generator=g) * 0.1, torch.rand(O, K, device=DEV, generator=g) * 0.1 + 0.01]
    p += [torch.randn(O, device=DEV, generator=g), torch.rand(O, device=DEV, generator=g) + 0.01] if bias else [None, None]
    dy = torch.randn(S, rows, O, device=DEV, generator=g)
    return BayesianLinear(K, O, S, 1000.0, bias=bias, seed=seed, weight_offset=8), x, p, dy


def _pass(layer, x, p, dy, step=3):
    leaves = [t.detach().requires_grad_() for t in [x] + [q for q in p if q is not None]]
    args = leaves[1:] + [None] * (4 - len(leaves[1:]))
    y = layer.forward(leaves[0], *args, step=step)
    return [y.detach()] + list(torch.autograd.grad(y, leaves, dy))


def _general(layer, x, p, dy, step=3):
    """The same pass through binding.py alone."""
    from paper_2604_04736_amd import binding as hot
    rows = x.shape[-2]
    rng = hot.hot_rng(layer.seed, step, layer.first_sample)
    y = torch.empty(S, rows, O, device=DEV)
    hot.hot_linear_forward_rng(rng, x, *p, y, layer.weight_offset, layer.bias_offset)
    grads = [torch.empty_like(q) if q is not None else None for q in p]
    dx = torch.empty(S, rows, K, device=DEV)
    n = hot.hot_linear_backward_workspace_bytes(rows, K, O, S)
    ws = torch.empty(n // 4, device=DEV) if n else None
    hot.hot_linear_backward_rng(rng, x, dy, *p, *grads, dx, S, 1000.0, hot.HOT_REDUCE_NONE, layer.weight_offset, layer.bias_offset, workspace=ws)
    return [y, dx if x.dim() == 3 else dx.sum(0)] + [g for g in grads if g is not None]


@pytest.mark.parametrize("rows", [1, 64, 200])
@pytest.mark.parametrize("own", [False, True])
@pytest.mark.parametrize("bias", [False, True])
def test_native_calls_are_the_general_path(rows, own, bias):
    layer, x, p, dy = _layer(rows, own, bias)
    want = _general(layer, x, p, dy)
    for got in (_pass(layer, x, p, dy), _pass(layer, x.transpose(-1, -2).contiguous().transpose(-1, -2), p, dy),
                _pass(layer, x, p, dy.transpose(1, 2).contiguous().transpose(1, 2))):
        assert len(got) == len(want) and all(torch.equal(a, b) for a, b in zip(got, want))
    # a strided weight: refused, as in binding.py
    with pytest.raises(TypeError):
        layer.forward(x, p[0].t().contiguous().t(), *p[1:], step=3)
    with pytest.raises(TypeError):
        layer.forward(x, p[0].double(), *p[1:], step=3)
    with pytest.raises(TypeError):
        layer.forward(x.cpu(), *[q.cpu() if q is not None else None for q in p], step=3)
    with pytest.raises((TypeError, ValueError)):
        layer.forward(x[..., :K - 4].contiguous(), *p, step=3)


def test_hooks_transforms_and_threads():
    layer, x, p, dy = _layer(64, True)
    want = _pass(layer, x, p, dy)
    with torch.autograd.graph.save_on_cpu():
        assert all(torch.equal(a, b) for a, b in zip(_pass(layer, x, p, dy), want))
    with pytest.raises(RuntimeError):              # (an autograd function without rules for them)
        torch.func.grad(lambda m: layer.forward(x, m, *p[1:], step=3).sum())(p[0])
    with pytest.raises(RuntimeError):
        torch.func.vmap(lambda v: layer.forward(v, *p, step=3))(torch.stack([x, x]))
    # a parameter changed between forward and backward is noticed
    m = p[0].clone().requires_grad_()
    y = layer.forward(x, m, *p[1:], step=3)
    with torch.no_grad():
        m.add_(1.0)
    with pytest.raises(RuntimeError):
        torch.autograd.grad(y, m, dy)
    # several threads, each with a stream of its own
    results, errors = [None] * 4, []

    def work(i):
        try:
            s = torch.cuda.Stream()
            s.wait_stream(torch.cuda.default_stream())
            with torch.cuda.stream(s):
                for _ in range(20):
                    results[i] = _pass(layer, x, p, dy)
            s.synchronize()
        except Exception as e:       # noqa: BLE001 (reported below)
            errors.append(e)
    torch.cuda.synchronize()
    threads = [threading.Thread(target=work, args=(i,)) for i in range(4)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not errors
    for r in results:
        assert all(torch.equal(a, b) for a, b in zip(r, want))


def test_statistics_of_what_the_native_call_leaves_to_the_general_path():
    from paper_2604_04736_amd import binding as hot
    y = torch.randn(5, 40, device=DEV)
    mean, std = torch.empty(33, device=DEV), torch.empty(33, device=DEV)
    hot.hot_stats_whole(y[:, :33], 1, mean, std)            # rows with a pitch
    want, want_std = torch.empty(33, device=DEV), torch.empty(33, device=DEV)
    hot.hot_stats_whole(y[:, :33].contiguous(), 1, want, want_std)
    assert torch.equal(mean, want) and torch.equal(std, want_std)
    assert torch.allclose(mean.double(), y[:, :33].double().mean(0), atol=1e-6)
    for bad in (mean.double(), mean[:32], mean.cpu()):
        with pytest.raises(TypeError):
            hot.hot_stats_whole(y[:, :33], 1, bad, std)
    with pytest.raises(hot.HotError):
        hot.hot_stats_whole(y, 5, torch.empty(40, device=DEV), torch.empty(40, device=DEV))      # ddof as large as the samples are many


@pytest.mark.parametrize("rows", [64, 200])
def test_parameters_of_another_size_than_the_layer_are_refused(rows):
    """Dense arrays that fit each other and not the layer: with more outputs than it has, its draws would run into those of its biases
    and of the next layer."""
    for height in (O + 30, O - 2):
        layer, x, p, _ = _layer(rows, True)
        g = torch.Generator(device=DEV).manual_seed(3)
        p = [torch.rand(height, K, device=DEV, generator=g), torch.rand(height, K, device=DEV, generator=g),
             torch.rand(height, device=DEV, generator=g), torch.rand(height, device=DEV, generator=g)]
        with pytest.raises(TypeError):
            layer.forward(x, *p, step=3)
    # another width: input gradients have the layer's
    layer, x, p, dy = _layer(rows, True)
    narrow = [t[..., :K - 4].contiguous() for t in (x, p[0], p[1])]
    with pytest.raises(TypeError):
        _pass(layer, narrow[0], narrow[1:] + p[2:], dy)


def test_sizes_and_seeds_of_any_integer_type():
    """NumPy's integers (a seed from a generator, a rank's first sample), as the ctypes calls take them."""
    import numpy as np
    from paper_2604_04736_amd.autograd import BayesianLinear
    layer, x, p, dy = _layer(64, True, seed=5)
    layer.first_sample = 6
    want = _pass(layer, x, p, dy)
    for kind in (np.int32, np.int64, np.uint64):
        other = BayesianLinear(kind(K), kind(O), kind(S), 1000.0, seed=kind(5), first_sample=kind(6), weight_offset=kind(8))
        assert all(torch.equal(a, b) for a, b in zip(_pass(other, x, p, dy, step=kind(3)), want))
    layer.seed = -(1 << 63)                     # (taken modulo 2^64, as ever)
    want = _pass(layer, x, p, dy)
    layer.seed = np.int64(-(1 << 63))
    assert all(torch.equal(a, b) for a, b in zip(_pass(layer, x, p, dy), want))
    layer.seed = 5.0
    with pytest.raises(TypeError):
        _pass(layer, x, p, dy)


@pytest.mark.parametrize("native", [True, False])
def test_without_room_for_the_scratch_a_layer_runs_as_without_it(native, monkeypatch):
    """Scratch memory for the drawn weights only buys time: where the allocator has none left the call is the one without."""
    from paper_2604_04736_amd import binding as hot
    from paper_2604_04736_amd.autograd import BayesianLinear
    r, k, o, s = 1024, 2048, 2048, 8
    mib = 1 << 20
    split = hot.hot_linear_backward_workspace_bytes(r, k, o, s)
    assert hot.hot_linear_planes_workspace_bytes(r, k, o, s, 0, True) >= 192 * mib and 128 * mib <= split <= 129 * mib
    assert hot.hot_linear_planes_workspace_bytes(r, k, o, s, 1) >= 192 * mib
    if not native:
        for name in ("linear_forward", "linear_backward"):
            monkeypatch.setattr(hot.host(), name, lambda *a: None)
    gc.collect()
    torch.cuda.empty_cache()                    # (so that what is made now leaves no room inside blocks of other tests)
    g = torch.Generator(device=DEV).manual_seed(1)
    x, dy = torch.randn(s, r, k, device=DEV, generator=g), torch.randn(s, r, o, device=DEV, generator=g)
    p = [torch.randn(o, k, device=DEV, generator=g) * 0.1, torch.rand(o, k, device=DEV, generator=g) * 0.1 + 0.01]
    layer, rng = BayesianLinear(k, o, s, 1000.0, bias=False, seed=5), hot.hot_rng(5, 3, 0)
    want = [torch.empty(s, r, o, device=DEV), torch.empty_like(x), torch.empty_like(p[0]), torch.empty_like(p[1])]
    hot.hot_linear_forward_rng(rng, x, *p, None, None, want[0])
    ws = torch.empty(split, dtype=torch.uint8, device=DEV)
    hot.hot_linear_backward_rng(rng, x, dy, *p, None, None, *want[2:], None, None, want[1], s, 1000.0, hot.HOT_REDUCE_NONE, workspace=ws)
    del ws
    leaves = [t.requires_grad_() for t in (x, *p)]

    def with_room(bytes_left, call):
        torch.cuda.synchronize()
        torch.cuda.empty_cache()
        torch.cuda.set_per_process_memory_fraction((torch.cuda.memory_reserved() + bytes_left) / torch.cuda.get_device_properties(0).total_memory)
        try:
            return call()
        finally:
            torch.cuda.set_per_process_memory_fraction(1.0)

    y = with_room((64 + 128) * mib, lambda: layer.forward(*leaves, None, None, step=3))
    got = [y.detach()] + list(with_room((64 + 32 + 160) * mib, lambda: torch.autograd.grad(y, leaves, dy, retain_graph=True)))
    assert all(torch.equal(a, b) for a, b in zip(got, want))
    del got
    with pytest.raises(torch.OutOfMemoryError):         # (no room for the scratch that the backward pass has always asked for)
        with_room((64 + 32 + 64) * mib, lambda: torch.autograd.grad(y, leaves, dy))
