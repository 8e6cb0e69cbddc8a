"""The product with weights that are drawn once into a workspace as bf16 pieces: y and dx are those of the call without a
workspace, whose kernel the oracle checks (test_parity_linear_gpu.py), bit for bit, since the products and their order are the same."""
import pytest
import torch

pytestmark = pytest.mark.gpu
DEV = "cuda"


@pytest.fixture(scope="module")
def hot():
    from paper_2604_04736_amd import binding
    return binding


def _inputs(seed, rows, k, o, s, own, ldx):
    g = torch.Generator(device=DEV).manual_seed(seed)
    x = torch.full((s, rows, ldx) if own else (rows, ldx), float("nan"), device=DEV)
    x[..., :k] = torch.randn(*x.shape[:-1], k, device=DEV, generator=g)
    return dict(x=x[..., :k], mu_w=torch.randn(o, k, device=DEV, generator=g) * (2.0 / k) ** 0.5,
                sigma_w=torch.rand(o, k, device=DEV, generator=g) * 0.1 + 1e-3, mu_b=torch.randn(o, device=DEV, generator=g),
                sigma_b=torch.rand(o, device=DEV, generator=g) + 0.01, dy=torch.randn(s, rows, o, device=DEV, generator=g) / rows)


def _workspace(bytes_):
    """The workspace with what lies behind it: all of it NaN in whatever pieces it is read."""
    whole = torch.full((bytes_ + 4096,), 255, dtype=torch.uint8, device=DEV)
    return whole, whole[:bytes_]


# (rows, in, out, samples, per-sample x, tile code): every tile, ragged rows, inputs (whole and half steps, odd and even numbers of
# them) and outputs
FORWARD = [(1460, 24, 769, 1, False, 11), (3031, 28, 125, 3, True, 11), (3968, 36, 937, 4, False, 13), (4864, 36, 724, 4, True, 13),
           (7718, 24, 985, 2, False, 21), (7911, 36, 555, 3, True, 21), (1101, 84, 2236, 3, False, 22), (6283, 236, 102, 4, True, 22),
           (4250, 84, 772, 3, False, 23), (5967, 212, 131, 4, True, 23), (2103, 148, 1472, 2, False, 31), (7468, 44, 507, 4, True, 31),
           (720, 148, 2771, 4, False, 33), (1484, 144, 1821, 3, True, 33)]


@pytest.mark.parametrize("rows,k,o,s,own,code", FORWARD)
def test_forward_with_drawn_weights_in_a_workspace(hot, rows, k, o, s, own, code):
    print("case planes forward", rows, k, o, s, own, code, flush=True)
    ldx = k + 4 if rows % 2 else k
    bytes_ = hot.hot_linear_planes_workspace_bytes(rows, k, o, s, 0, own)
    assert hot.hot_linear_planes_shape(rows, k, o, s, 0, own, ldx=ldx, workspace_bytes=bytes_) == code
    assert hot.hot_linear_planes_shape(rows, k, o, s, 0, own, ldx=ldx, workspace_bytes=bytes_ - 16) == 0
    t = _inputs(rows + k, rows, k, o, s, own, ldx)
    rng = hot.hot_rng(seed=0xABCDEF12345, step=4, first_sample=2 * s)
    w_off, b_off = 4 * 1000, 4 * 1000 + (o * k + 3) // 4 * 4 + 8

    def run(ws, bias=True):
        y = torch.full((s, rows, o), float("nan"), device=DEV)
        b = (t["mu_b"], t["sigma_b"]) if bias else (None, None)
        hot.hot_linear_forward_rng(rng, t["x"], t["mu_w"], t["sigma_w"], *b, y, w_off, b_off, workspace=ws)
        return y

    for bias in (True, False):
        want = run(None, bias)
        assert torch.isfinite(want).all()
        whole, ws = _workspace(bytes_)
        assert torch.equal(run(ws, bias), want)
        assert (whole[bytes_:] == 255).all()
    whole, ws = _workspace(bytes_)
    assert torch.equal(run(ws[:-16]), run(None)) and (whole == 255).all()            # too small: not used
    # infinities, NaN and values beyond the largest bf16 number
    for at, bad in ((0, float("inf")), (rows // 2, 3.4e38), (rows - 1, float("nan"))):
        (t["x"][-1] if own else t["x"])[at, k - 1] = bad
    t["mu_w"][o - 1, 0] = float("-inf")
    assert torch.allclose(run(_workspace(bytes_)[1]), run(None), rtol=0.0, atol=0.0, equal_nan=True)


# (rows, in, out, samples, tile code)
BACKWARD = [(8924, 64, 84, 2, 11), (4995, 1412, 36, 2, 13), (8772, 444, 24, 4, 21), (5499, 1104, 100, 1, 22), (1060, 2688, 56, 4, 23),
            (8200, 388, 36, 4, 31), (7898, 1080, 140, 1, 33)]


@pytest.mark.parametrize("rows,k,o,s,code", BACKWARD)
def test_input_gradients_with_drawn_weights_in_a_workspace(hot, rows, k, o, s, code):
    print("case planes input gradients", rows, k, o, s, code, flush=True)
    bytes_ = max(hot.hot_linear_backward_workspace_bytes(rows, k, o, s), hot.hot_linear_planes_workspace_bytes(rows, k, o, s, 1))
    assert hot.hot_linear_planes_shape(rows, k, o, s, 1, workspace_bytes=bytes_) == code
    t = _inputs(rows + k, rows, k, o, s, True, k)
    rng = hot.hot_rng(seed=0xABCDEF12345, step=4, first_sample=s)

    def run(ws):
        grads = [torch.full_like(t[name], float("nan")) for name in ("mu_w", "sigma_w", "mu_b", "sigma_b")]
        dx = torch.full((s, rows, k), float("nan"), device=DEV)
        hot.hot_linear_backward_rng(rng, t["x"], t["dy"], t["mu_w"], t["sigma_w"], t["mu_b"], t["sigma_b"], *grads, dx, s, 50000.0,
                                    hot.HOT_REDUCE_NONE, 4000, 4000 + o * k, workspace=ws)
        return grads, dx

    grads, want = run(None)
    whole, ws = _workspace(bytes_)
    got, dx = run(ws)
    assert torch.isfinite(want).all() and torch.equal(dx, want)
    assert (whole[bytes_:] == 255).all()
    for a, b in zip(got, grads):        # (with a workspace the weight gradients may add up their rows in parts)
        assert torch.isfinite(a).all() and (a - b).norm() <= 1e-5 * b.norm()
    t["dy"][0, 0, 0] = float("inf")
    assert torch.allclose(run(_workspace(bytes_)[1])[1], run(None)[1], rtol=0.0, atol=0.0, equal_nan=True)


def test_the_layer_hands_over_a_workspace(hot):
    """BayesianLinear on a layer of thousands of rows: y, dx and the gradients are those of the calls with workspaces."""
    from paper_2604_04736_amd.autograd import BayesianLinear
    rows, k, o, s = 16640, 192, 768, 2
    assert hot.hot_linear_planes_shape(rows, k, o, s, 0, True) and hot.hot_linear_planes_shape(rows, k, o, s, 1)
    t = _inputs(1, rows, k, o, s, True, k)
    layer = BayesianLinear(k, o, s, 50000.0, seed=77)
    leaves = [t[n].requires_grad_() for n in ("x", "mu_w", "sigma_w", "mu_b", "sigma_b")]
    y = layer.forward(*leaves, step=3)
    dx = torch.autograd.grad(y, leaves, t["dy"])[0]
    rng = hot.hot_rng(seed=77, step=3, first_sample=0)
    want = torch.empty_like(y)
    d = [v.detach() for v in leaves]
    hot.hot_linear_forward_rng(rng, *d, want, 0, o * k)
    assert torch.equal(y.detach(), want)
    want_dx = torch.empty_like(dx)
    hot.hot_linear_backward_rng(rng, d[0], t["dy"], *d[1:], *[torch.empty_like(v) for v in d[1:]], want_dx, s, 50000.0, hot.HOT_REDUCE_NONE, 0, o * k)
    assert torch.equal(dx, want_dx)


@pytest.mark.parametrize("k,o,bias", [(4, 1, True), (4, 1, False), (128, 128, True), (96, 131, True), (1024, 63, True), (16384, 4, False),
                                      (16384, 4, True), (2048, 33, True)])
def test_kl_of_a_layer_in_one_launch(hot, k, o, bias):
    """Up to HOT_KL_LAYER_MAX parameters (the first six; then the two sums of hot_kl): against fp64."""
    from paper_2604_04736_amd.autograd import BayesianLinear
    one_launch = k * o + (o if bias else 0) <= hot.HOT_KL_LAYER_MAX
    g = torch.Generator(device=DEV).manual_seed(k + o)
    mu_w, sigma_w = torch.randn(o, k, device=DEV, generator=g), torch.rand(o, k, device=DEV, generator=g) + 0.01
    mu_b, sigma_b = torch.randn(o, device=DEV, generator=g), torch.rand(o, device=DEV, generator=g) + 0.01
    layer = BayesianLinear(k, o, 1, 100.0, bias=bias)
    got = layer.kl(mu_w, sigma_w, mu_b if bias else None, sigma_b if bias else None)
    assert hasattr(layer, "_kl_plans") != one_launch and got.shape == () and got.dtype == torch.float64
    terms = [(m.double() ** 2, s.double() ** 2) for m, s in [(mu_w, sigma_w)] + ([(mu_b, sigma_b)] if bias else [])]
    want = sum(0.5 * (s + m - 1.0 - s.log()).sum() for m, s in terms)
    size = sum(0.5 * (s + m + 1.0 + s.log().abs()).sum() for m, s in terms)
    # (the hardware's log2 is within 6e-8 of a number in [1/2, 1): 8e-8 of each addend's ln sigma^2)
    assert abs(got.item() - want.item()) <= 1e-7 * size.item()
    # a flat view and a strided one: as before
    assert abs(layer.kl(mu_w.reshape(-1), sigma_w.reshape(-1), mu_b, sigma_b).item() - got.item()) <= 1e-12 * size.item()
    strided = mu_w.t().contiguous().t()
    assert abs(layer.kl(strided, sigma_w, mu_b, sigma_b).item() - got.item()) <= 1e-12 * size.item()
    if one_launch:
        sigma_w[0, 0] = 0.0
        assert layer.kl(mu_w, sigma_w, mu_b, sigma_b).item() == float("inf")
        sigma_w[0, 0] = -1.0
        assert layer.kl(mu_w, sigma_w, mu_b, sigma_b).isnan()


@pytest.mark.parametrize("rows,k,o,s,own", [(16, 2048, 2048, 2, True), (3, 2048, 2049, 2, False), (16, 5000, 1100, 4, True), (9, 5000, 1100, 4, False),
                                            (16, 2048, 1400, 3, True), (16, 1024, 700, 7, False), (1, 700, 1200, 16, True), (16, 2048, 2240, 2, True)])
def test_samples_in_workgroups_of_their_own(hot, rows, k, o, s, own):
    """Few rows, sixteen waves to a tile: up to one workgroup per compute unit the samples are dealt out; every sample's y is that of a call
    with it alone, bit for bit (the last layer is beyond the line)."""
    print("case dealt samples", rows, k, o, s, own, flush=True)
    t = _inputs(rows + k + o, rows, k, o, s, own, k)

    def run(x, first, n):
        y = torch.full((n, rows, o), float("nan"), device=DEV)
        hot.hot_linear_forward_rng(hot.hot_rng(seed=3, step=1, first_sample=first), x, t["mu_w"], t["sigma_w"], t["mu_b"], t["sigma_b"], y, 0, o * k)
        return y

    y = run(t["x"], 5, s)
    for i in range(s):
        assert torch.equal(y[i], run(t["x"][i].contiguous() if own else t["x"], 5 + i, 1)[0])
