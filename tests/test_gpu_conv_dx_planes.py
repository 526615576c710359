"""A convolution's dX product takes its fp32 weights exactly, whatever their range: in three bf16 planes that add up to them, in every kernel and entry point.

One nonzero code of +-1 per image and a step size of 1 make every element of dX one weight (or zero) as the planes hold it, so the expected value is the
weight itself, bit for bit.  Random mantissas fill all 24 bits of a weight, and weights far below their channel's largest have to keep theirs.
"""
import numpy as np
import pytest
import torch  # noqa: F401  (before the library: both bring a HIP runtime, and the first one in serves both)

pytestmark = pytest.mark.gpu

# every tile of both kernels: conv_dx_kernel (waves 0) and conv_dx_split_kernel; a partial block of 32 channels, K that ends inside a group of 8, planes
# that are copied to whole dwords (odd ones)
FORMS = [((33, 33, 33, 30, 115), (0, 2)), ((90, 33, 28, 28, 115), (0, 4)), ((61, 130, 28, 28, 115), (0, 7)), ((33, 33, 14, 14, 115), (4, 2)),
         ((90, 33, 14, 14, 115), (4, 4)), ((90, 130, 13, 13, 115), (4, 7)), ((1, 33, 3, 3, 114), (8, 2)), ((90, 33, 9, 9, 520), (8, 4)),
         ((90, 33, 13, 13, 520), (8, 7))]


def _weights(rng, K, C, what):
    W = (rng.standard_normal((K, C, 3, 3)) * 0.02).astype(np.float32)
    if what == "channel scales":                       # each channel has a scale of its own
        W *= np.float32(2.0) ** rng.integers(-40, 41, size=(1, C, 1, 1)).astype(np.float32)
        W[:, C // 2] = 0
    elif what == "outlier":                            # one output channel's weights 2^15 to 2^25 above the others: these keep all their bits
        W[K // 2] *= np.float32(2.0) ** rng.integers(15, 26, size=(C, 1, 1)).astype(np.float32)
    elif what == "tiny":                               # one weight 2^-30 of its channel's largest
        W[K // 2, C - 1, 1, 1] = 2.0 ** -30 * np.abs(W[:, C - 1]).max()
    elif what == "huge":
        W *= np.float32(2.0 ** 110)
    elif what == "small":
        W *= np.float32(2.0 ** -110)
    elif what in ("inf", "nan"):
        W[K - 1, C // 2, 2, 0] = np.float32(what)
    return W


def _run(W, N, H, Wd, entry, rng):
    import paper_2004_04729_amd as dbp
    from gpu_util import DEV, dev, stream
    K, C = W.shape[:2]
    at = [(int(rng.integers(K)), int(rng.integers(H)), int(rng.integers(Wd)), int(rng.choice([-1, 1]))) for _ in range(N)]
    delta = np.zeros((N, K, H, Wd), np.float32)
    for n, (k, h, w, m) in enumerate(at):
        delta[n, k, h, w] = m
    d, Wt = dev(delta), dev(W)
    codes = torch.empty(delta.shape, dtype=torch.int8, device=DEV)
    dX = torch.full((N, C, H, Wd), 7.0, dtype=torch.float32, device=DEV)
    dims = (N, C, H, Wd, K, 3, 3, 1, 1)
    ws = torch.empty(dbp.conv2d_workspace_bytes(*dims), dtype=torch.uint8, device=DEV)
    if entry == "backward":
        dbp.dithered_conv2d_backward(d, Wt, None, dbp.F32, *dims, 1.0, 3, 0, codes, dX, None, ws, None, dbp.PATH_MFMA, stream())
    else:
        dbp.nsd_quantize(d, N * K, H * Wd, 1.0, 3, 0, codes, None, None, stream())
        dbp.conv2d_products(codes, None, 1.0, Wt, None, dbp.F32, *dims, dX, None, ws, dbp.PATH_MFMA, stream())
    torch.cuda.synchronize()
    assert np.array_equal(codes.cpu().numpy(), delta.astype(np.int8))
    return at, dX.cpu().numpy()


def _expected(W, at, N, C, H, Wd):
    out = np.zeros((N, C, H + 2, Wd + 2))
    for n, (k, h, w, m) in enumerate(at):
        out[n, :, h:h + 3, w:w + 3] = m * W[k].astype(np.float64)
    return out[:, :, 1:-1, 1:-1]


@pytest.mark.parametrize("what", ["normal", "channel scales", "outlier", "tiny", "huge", "small", "inf", "nan"])
@pytest.mark.parametrize("case,form", FORMS)
def test_conv_dx_weights_are_exact(case, form, what):
    from plan_util import conv_dx_kernel
    N, C, H, Wd, K = case
    assert conv_dx_kernel(N, C, H, Wd, K, 3, 3, 1, 1) == form
    rng = np.random.default_rng(N + C + K)
    W = _weights(rng, K, C, what)
    at, got = _run(W, N, H, Wd, "backward", rng)
    finite = [c for c in range(C) if np.isfinite(W[:, c]).all()]            # (0 * inf is a NaN: a channel with one has no other elements where its tap reaches)
    step = 2.0 ** -133 if what == "small" else 0.0                           # the smallest bf16: what truncating the last plane can lose
    assert np.all(np.abs(got[:, finite] - _expected(W, at, N, C, H, Wd)[:, finite]) <= step)
    assert len(finite) == C or not np.isfinite(got[:, C // 2]).all()


@pytest.mark.parametrize("case", [(61, 130, 28, 28, 115), (33, 33, 14, 14, 115), (4, 33, 9, 9, 113), (90, 130, 13, 13, 115)])
def test_conv_dx_weights_are_exact_in_products_alone(case):
    N, C, H, Wd, K = case
    rng = np.random.default_rng(11)
    W = _weights(rng, K, C, "outlier")
    at, got = _run(W, N, H, Wd, "products", rng)
    assert np.array_equal(got, _expected(W, at, N, C, H, Wd))


@pytest.mark.parametrize("what", ["normal", "outlier"])
def test_conv_dx_weights_are_exact_in_a_layer_call(what):
    """The whole-layer entry point: the same dX, bit for bit, as the products of its codes and its step size."""
    import paper_2004_04729_amd as dbp
    from gpu_util import DEV, dev, stream, check_products
    from oracle import oracle as O
    N, C, H, Wd, K = 5, 33, 9, 9, 130
    rng = np.random.default_rng(2)
    W = _weights(rng, K, C, what)
    delta = rng.laplace(0, 1e-3, size=(N, K, H, Wd)).astype(np.float32)
    act = rng.standard_normal(delta.shape).astype(np.float32)
    X = np.maximum(rng.standard_normal((N, C, H, Wd)), 0).astype(np.float32)
    dims = (N, C, H, Wd, K, 3, 3, 1, 1)
    codes = torch.empty(delta.shape, dtype=torch.int8, device=DEV)
    dX = torch.empty(X.shape, dtype=torch.float32, device=DEV)
    dW = torch.empty(W.shape, dtype=torch.float32, device=DEV)
    step = torch.empty(2, dtype=torch.float32, device=DEV)
    ws = torch.empty(dbp.conv2d_layer_workspace_bytes(*dims), dtype=torch.uint8, device=DEV)
    dbp.dithered_conv2d_layer_backward(dev(delta), dev(act), dev(W), dev(X), dbp.F32, *dims, 4.0, 9, 0, codes, dX, dW, None, step, ws, None,
                                       dbp.PATH_AUTO, stream())
    torch.cuda.synchronize()
    alone = torch.empty_like(dX)
    dbp.conv2d_products(codes, None, float(step[0]), dev(W), None, dbp.F32, *dims, alone, None, ws, dbp.PATH_MFMA, stream())
    torch.cuda.synchronize()
    assert torch.equal(dX, alone)
    k = codes.cpu().numpy()
    kw = dict(stride=1, pad=1)
    rX, rW, _ = O.conv2d_backward(W, X, codes=k, step=float(step[0]), **kw)
    aX, aW, _ = O.conv2d_backward(np.abs(W), X, codes=np.abs(k), step=float(step[0]), **kw)
    check_products(dX.cpu().numpy(), rX, aX, "dX")
    check_products(dW.cpu().numpy(), rW, aW, "dW")
