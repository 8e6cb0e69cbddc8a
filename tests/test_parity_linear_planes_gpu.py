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
FORWARD = [(8542, 24, 128, 2, False, 11), (1463, 84, 392, 2, True, 11), (1285, 84, 2177, 3, False, 13), (1320, 324, 752, 3, True, 13),
           (8140, 32, 388, 4, False, 21), (5469, 52, 1093, 2, True, 21), (853, 84, 2925, 3, False, 22), (8470, 296, 101, 3, True, 22),
           (4626, 216, 326, 3, False, 23), (1820, 60, 2050, 3, True, 23), (8759, 124, 293, 3, False, 31), (6933, 348, 202, 3, True, 31),
           (2236, 168, 1179, 3, False, 33), (7240, 228, 370, 3, True, 33),
           # tiles of 256 x 256, and planes beyond 256 MiB
           (8901, 644, 657, 2, True, 44), (1184, 636, 3421, 3, True, 44), (462, 1604, 7070, 4, False, 44), (368, 2828, 7969, 2, False, 23)]


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
BACKWARD = [(6854, 916, 20, 2, 11), (519, 2328, 392, 4, 13), (820, 1032, 232, 4, 21), (555, 2140, 244, 3, 22), (7092, 148, 276, 4, 23),
            (8800, 112, 344, 4, 31), (3643, 1128, 212, 2, 33),
            (479, 6320, 636, 4, 44), (441, 7672, 1604, 4, 44), (332, 6024, 2048, 4, 33)]


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


# The layers of the kernel for tens to hundreds of rows (tile code + 100): two accumulators to a sum
APART = [(646, 128, 1395, 2, False, 111), (150, 148, 2779, 3, True, 111), (564, 140, 2833, 3, False, 113), (3475, 956, 168, 4, True, 113),
         (4389, 136, 231, 3, False, 122), (6012, 1020, 68, 4, True, 122), (1349, 316, 797, 4, False, 123), (4846, 664, 146, 4, True, 123)]


@pytest.mark.parametrize("rows,k,o,s,own,code", APART)
def test_forward_with_the_small_products_apart(hot, rows, k, o, s, own, code):
    """Against fp64 products of the library's own w, and no farther from them than the kernel that runs without a workspace; infinities, NaN
    and values beyond the largest bf16 number give what they give there."""
    print("case planes apart", rows, k, o, s, own, code, flush=True)
    ldx = k + 4 if rows % 2 else k
    bytes_ = hot.hot_linear_planes_workspace_bytes(rows, k, o, s, 0, own)
    assert hot.hot_linear_planes_shape(rows, k, o, s, 0, own, ldx=ldx, workspace_bytes=bytes_) == code
    assert hot.hot_linear_kernel_shape(rows, k, o, s, 0, own, ldx=ldx) > 0
    t = _inputs(rows + k, rows, k, o, s, own, ldx)
    rng = hot.hot_rng(seed=0xABCDEF12345, step=4, first_sample=2 * s)
    plan = hot.hot_create(o * k, o * k, s, s, 1000.0, 0)
    w = torch.empty(s, o * k, device=DEV)
    hot.hot_forward_rng(plan, rng, t["mu_w"].reshape(-1), t["sigma_w"].reshape(-1), w, torch.empty(1, dtype=torch.float64, device=DEV))
    b_off = (o * k + 3) // 4 * 4 + 8

    def run(ws):
        y = torch.full((s, rows, o), float("nan"), device=DEV)
        hot.hot_linear_forward_rng(rng, t["x"], t["mu_w"], t["sigma_w"], None, None, y, 0, 0, workspace=ws)
        return y

    plain = run(None)
    whole, ws = _workspace(bytes_)
    got = run(ws)
    assert (whole[bytes_:] == 255).all()
    x64 = t["x"].double().expand(s, rows, k) if not own else t["x"].double()
    want = torch.stack([x64[i] @ w[i].view(o, k).double().t() for i in range(s)])
    size = torch.stack([x64[i].abs() @ w[i].view(o, k).double().abs().t() for i in range(s)])
    # one rounding of the large products and five of the small ones to sixteen indices, below 2^-24 of the magnitude sum each at most, and what
    # the pieces leave out of a product, 3 * 2^-24
    assert ((got.double() - want).abs() <= (k / 16 + 8) * 2.0 ** -24 * size).all()
    assert (got.double() - want).norm() <= 0.9 * (plain.double() - want).norm()
    # with biases: the same sums, one rounding more
    y = torch.empty_like(got)
    hot.hot_linear_forward_rng(rng, t["x"], t["mu_w"], t["sigma_w"], t["mu_b"], t["sigma_b"], y, 0, b_off, workspace=ws)
    zero = torch.zeros(s, rows, o, device=DEV)
    hot.hot_linear_forward_rng(rng, torch.zeros_like(t["x"]), t["mu_w"], t["sigma_w"], t["mu_b"], t["sigma_b"], zero, 0, b_off)
    assert torch.equal(y, got + zero[:, :1])
    for at, bad in ((0, float("inf")), (rows // 2, 3.4e38), (rows - 1, float("nan"))):
        (t["x"][-1] if own else t["x"])[at, k - 1] = bad
    t["mu_w"][o - 1, 0] = float("-inf")
    got, plain = run(ws), run(None)
    assert torch.equal(got.isnan(), plain.isnan()) and torch.equal(got.isinf(), plain.isinf())
    assert torch.equal(got[got.isinf()], plain[plain.isinf()])
    finite = torch.isfinite(got)
    assert torch.allclose(got[finite], plain[finite], rtol=1e-3, atol=1e-3)


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


@pytest.mark.parametrize("n_w,n_b", [(1, 0), (7, 3), (4096, 1), (65533, 3), (65536, 0)])
def test_kl_of_arrays_on_any_four_byte_boundary(hot, n_w, n_b):
    g = torch.Generator(device=DEV).manual_seed(n_w + n_b)
    flat = torch.rand(2 * (n_w + n_b) + 5, device=DEV, generator=g) + 0.01
    at, parts = 1, []
    for n in (n_w, n_w, n_b, n_b):
        parts.append(flat[at:at + n] if n else None)
        at += n + 1
    out = torch.full((3,), -1.0, dtype=torch.float64, device=DEV)
    hot.hot_kl_layer(*parts, out[1:2])
    v = torch.cat([q for q in (parts[0], parts[2]) if q is not None]).double(), torch.cat([q for q in (parts[1], parts[3]) if q is not None]).double()
    want, size = (0.5 * (v[1] ** 2 + v[0] ** 2 + i - 2.0 * f(v[1].log())).sum() for i, f in ((-1.0, lambda t: t), (1.0, lambda t: -t.abs())))
    assert abs(out[1].item() - want.item()) <= 1e-7 * size.item()          # (as above)
    assert out[0].item() == -1.0 and out[2].item() == -1.0


def test_kl_of_a_layer_refuses_what_it_cannot_take(hot):
    t, out = torch.ones(65537, device=DEV), torch.zeros(1, dtype=torch.float64, device=DEV)
    for mu_w, sigma_w, mu_b, sigma_b, code in ((t, t, None, None, hot.HOT_ERANGE), (t[:65536], t[:65536], t[:1], t[:1], hot.HOT_ERANGE),
                                               (t[:0], t[:0], None, None, hot.HOT_EINVAL)):
        with pytest.raises(hot.HotError) as e:
            hot.hot_kl_layer(mu_w, sigma_w, mu_b, sigma_b, out)
        assert e.value.code == code
    for args, error in (((t[:4], t[:4], t[:1], None, out), ValueError), ((t[:4], t[:8:2], None, None, out), TypeError),
                        ((t[:4], t[:4], None, None, out.float()), TypeError), ((t[:4].double(), t[:4], None, None, out), TypeError)):
        with pytest.raises(error):
            hot.hot_kl_layer(*args)


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
