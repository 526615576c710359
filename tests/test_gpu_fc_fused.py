"""Fully connected calls with few gradients (one launch, every workgroup quantises for itself) against the same work piece by piece: step size,
quantiser and products through their own entry points, whose kernels the other tests hold to the oracle.  Every output is the same bit for bit."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

# n = B * out: one gradient, a full level of the step size's tree and one more, the most that a fused call takes (and one call beyond it), rows
# shorter than a window of the reduction, widths that no vector divides, a reduction split over workgroups (partial sums in a second launch), bias columns
# that many threads share, that threads do not divide, and more of them than threads
SIZES = [(1, 5, 2), (2, 64, 1), (16, 100, 1), (17, 100, 1), (64, 100, 10), (16, 33, 16), (257, 70, 1), (27, 2592, 8), (3, 130, 85), (31, 515, 132), (4096, 64, 1),
         (512, 4096, 8), (16, 4100, 256), (64, 784, 64), (241, 77, 17), (64, 300, 128), (32, 72, 256), (2731, 70, 3), (8192, 64, 1),
         (2730, 70, 3), (4096, 64, 2), (1365, 40, 6), (24, 64, 341), (13, 64, 630), (2, 64, 513), (1, 70, 8192)]


def _delta(rng, B, out, odd):
    d = rng.laplace(0, 1e-3, size=(B, out)).astype(np.float32)
    if odd:                                             # saturated, infinite and not a number
        flat = d.reshape(-1)
        for i, v in enumerate((1.0, -1.0, np.inf, -np.inf, np.nan)):
            flat[(i * 37) % flat.size] = v
    return d


def _pieces(dbp, d, act, W, X, xd, B, in_, out, pair, step, q8, stream):
    """Codes, statistics, column sums and products of the separate entry points."""
    dev = d.device
    codes = torch.empty((B, out), dtype=torch.int8, device=dev)
    L = dbp.format_layout(B, out)
    fmt = torch.empty(L["total_bytes"], dtype=torch.uint8, device=dev)
    st = torch.zeros(32, dtype=torch.uint8, device=dev)
    dbp.nsd_quantize_ex(d, B, out, step, 7, 12345678901, codes, fmt, st, act=act, step_dev=pair, stream=stream)
    if q8:
        q, w, x = codes.cpu().numpy().astype(np.int64), W.cpu().numpy().astype(np.int64), X.cpu().numpy().astype(np.int64)
        return codes, st, torch.from_numpy((q @ w).astype(np.int32)), torch.from_numpy((q.T @ x).astype(np.int32))
    dX = torch.empty((B, in_), dtype=torch.float32, device=dev)
    dW = torch.empty((out, in_), dtype=torch.int32 if xd == dbp.I8 else torch.float32, device=dev)
    ws = torch.empty(dbp.linear_workspace_bytes(B, in_, out, xd), dtype=torch.uint8, device=dev)
    dbp.linear_products(codes, None, float(pair[0]) if pair is not None else step, W, X, xd, B, in_, out, dX, dW, ws, dbp.PATH_MFMA, stream)
    return codes, st, dX, dW


@pytest.mark.parametrize("odd", [False, True])
@pytest.mark.parametrize("mode", ["plain", "int8 activations", "q8", "layer", "layer without activations"])
@pytest.mark.parametrize("B,in_,out", SIZES)
def test_fused_call_equals_its_pieces(B, in_, out, mode, odd):
    import paper_2004_04729_amd as dbp
    from gpu_util import DEV, dev, stream
    rng = np.random.default_rng(B * 7 + in_ + out)
    layer, q8 = mode.startswith("layer"), mode == "q8"
    if layer and odd and B * out < 3:
        pytest.skip("a step size needs finite gradients")
    xd = dbp.I8 if q8 or mode == "int8 activations" else dbp.F32
    d = dev(_delta(rng, B, out, odd and not layer))
    act = dev(np.where(rng.random((B, out)) < 0.5, 0, rng.standard_normal((B, out))).astype(np.float32)) if mode == "layer" else None
    if layer and odd:                                   # saturation by one large gradient is what a finite tensor can have
        d.view(-1)[0] = 10.0
    W = dev(rng.integers(-127, 128, (out, in_)).astype(np.int8)) if q8 else dev(rng.standard_normal((out, in_)).astype(np.float32))
    X = dev(rng.integers(0, 128, (B, in_)).astype(np.int8)) if xd == dbp.I8 else dev(np.maximum(rng.standard_normal((B, in_)), 0).astype(np.float32))
    codes = torch.full((B, out), 99, dtype=torch.int8, device=DEV)
    dX = torch.full((B, in_), -7, dtype=torch.int32 if q8 else torch.float32, device=DEV)
    dW = torch.full((out, in_), -7, dtype=torch.int32 if xd == dbp.I8 else torch.float32, device=DEV)
    st = torch.full((32,), 0xEE, dtype=torch.uint8, device=DEV)
    step, pair, db = float(np.float32(5e-3)), None, None
    if layer:
        ws = torch.empty(dbp.linear_layer_workspace_bytes(B, in_, out, xd), dtype=torch.uint8, device=DEV)
        got_pair, db = torch.empty(2, dtype=torch.float32, device=DEV), torch.full((out,), 5.0, dtype=torch.float32, device=DEV)
        dbp.dithered_linear_layer_backward(d, act, W, X, xd, B, in_, out, 3.0, 7, 12345678901, codes, dX, dW, db, got_pair, ws, st, dbp.PATH_AUTO, stream())
        pair = torch.empty(2, dtype=torch.float32, device=DEV)
        dbp.step_size(d, act, B * out, 3.0, pair, torch.empty(dbp.step_size_workspace_bytes(B * out), dtype=torch.uint8, device=DEV), stream())
        assert torch.equal(got_pair, pair)
    else:
        ws = torch.empty(dbp.linear_workspace_bytes(B, in_, out, xd), dtype=torch.uint8, device=DEV)
        if q8:
            dbp.dithered_linear_backward_q8(d, W, X, B, in_, out, step, 7, 12345678901, codes, dX, dW, ws, st, stream())
        else:
            dbp.dithered_linear_backward(d, W, X, xd, B, in_, out, step, 7, 12345678901, codes, dX, dW, ws, st, dbp.PATH_AUTO, stream())
    torch.cuda.synchronize()
    if layer and float(pair[0]) == 0.0:                 # a degenerate tensor: zero codes, zero products
        assert not codes.any() and not dX.any() and not dW.any() and not db.any()
        return
    rc, rs, rX, rW = _pieces(dbp, d, act, W, X, xd, B, in_, out, pair, step, q8, stream())
    torch.cuda.synchronize()
    assert torch.equal(codes, rc) and torch.equal(st, rs)
    assert torch.equal(dX.cpu(), rX.cpu()) and torch.equal(dW.cpu(), rW.cpu())
    if db is not None:
        want = (np.float64(float(pair[0])) * codes.cpu().numpy().astype(np.int64).sum(axis=0)).astype(np.float32)
        assert np.array_equal(db.cpu().numpy(), want)


def test_results_in_the_place_of_the_gradients():
    """dX over delta (in = out): the quantiser has to be through before the products begin."""
    import paper_2004_04729_amd as dbp
    from gpu_util import DEV, dev, stream
    rng = np.random.default_rng(1)
    B, n = 64, 64
    d, W, X = rng.laplace(0, 1e-3, (B, n)).astype(np.float32), dev(rng.standard_normal((n, n)).astype(np.float32)), dev(rng.standard_normal((B, n)).astype(np.float32))
    ws = torch.empty(dbp.linear_workspace_bytes(B, n, n), dtype=torch.uint8, device=DEV)
    out = []
    for place in (False, True):
        delta, codes, dW = dev(d), torch.empty((B, n), dtype=torch.int8, device=DEV), torch.empty((n, n), dtype=torch.float32, device=DEV)
        dX = delta if place else torch.empty((B, n), dtype=torch.float32, device=DEV)
        dbp.dithered_linear_backward(delta, W, X, dbp.F32, B, n, n, 5e-3, 3, 0, codes, dX, dW, ws, None, dbp.PATH_AUTO, stream())
        torch.cuda.synchronize()
        out.append((codes, dX, dW))
    assert all(torch.equal(a, b) for a, b in zip(*out))


# One launch or launches of their own: the most gradients, kernels other than the direct one (a single output), and, by mode, the most workgroups of the
# products beside the one that writes what the quantiser leaves (in brackets)
@pytest.mark.parametrize("B,in_,out,mode,fused", [
    (64, 100, 10, "plain", True), (64, 100, 10, "layer", True), (64, 100, 10, "q8", True),
    (64, 64, 128, "plain", True), (64, 64, 128, "layer", True), (64, 64, 128, "q8", True),
    (64, 64, 129, "plain", False), (2731, 70, 3, "layer", False), (64, 64, 129, "q8", False), (16, 100, 1, "layer", False),
    (52, 8069, 106, "layer", True), (16, 8192, 500, "layer", False), (16, 8192, 500, "plain", True),         # [254], [256]
    (128, 65536, 32, "layer", True), (5, 83989, 367, "layer", False),                                        # 4096 gradients and fewer: [384], [1151]
    (64, 32768, 96, "q8", True), (64, 131072, 96, "q8", False), (183, 89604, 21, "q8", True), (9, 56482, 389, "q8", False),   # [160], [640], [614], [830]
    (64, 146865, 123, "int8 activations", False), (16, 65536, 500, "plain", True), (16, 131072, 500, "plain", False)])        # [861], [1152], [2304]
def test_one_launch_where_it_is_the_faster(B, in_, out, mode, fused):
    import paper_2004_04729_amd as dbp
    from gpu_util import DEV, graph_nodes
    layer, q8 = mode == "layer", mode == "q8"
    xd = dbp.I8 if q8 or mode == "int8 activations" else dbp.F32
    buf = lambda shape, dt: torch.zeros(shape, dtype=dt, device=DEV)
    d, W, X = buf((B, out), torch.float32), buf((out, in_), torch.int8 if q8 else torch.float32), buf((B, in_), torch.int8 if xd == dbp.I8 else torch.float32)
    codes, dX, dW = buf((B, out), torch.int8), buf((B, in_), torch.float32), buf((out, in_), torch.float32)
    pair, db = buf(2, torch.float32), buf(out, torch.float32)
    ws = buf(max(dbp.linear_layer_workspace_bytes(B, in_, out, xd), dbp.linear_workspace_bytes(B, in_, out, xd)), torch.uint8)

    def call(s):
        if layer:
            dbp.dithered_linear_layer_backward(d, d, W, X, xd, B, in_, out, 3.0, 7, 0, codes, dX, dW, db, pair, ws, None, dbp.PATH_AUTO, s)
        elif q8:
            dbp.dithered_linear_backward_q8(d, W, X, B, in_, out, 5e-3, 7, 0, codes, dX, dW, ws, None, s)
        else:
            dbp.dithered_linear_backward(d, W, X, xd, B, in_, out, 5e-3, 7, 0, codes, dX, dW, ws, None, dbp.PATH_AUTO, s)
    assert (graph_nodes(call) == 1) == fused


@pytest.mark.parametrize("bad", [np.inf, -np.inf, np.nan])
@pytest.mark.parametrize("masked", [False, True])
@pytest.mark.parametrize("B,in_,out", [(64, 100, 10), (64, 64, 128), (27, 2592, 8)])
def test_layer_call_with_a_gradient_that_is_no_number(B, in_, out, masked, bad):
    """No step size: zero codes, products and bias gradient, and the statistics count it; behind the rectifier's mask it is nothing at all."""
    import paper_2004_04729_amd as dbp
    from gpu_util import DEV, dev, stream
    rng = np.random.default_rng(3)
    d, act = _delta(rng, B, out, False), rng.standard_normal((B, out)).astype(np.float32)
    d[B // 2, out // 2], act[B // 2, out // 2] = bad, -1.0 if masked else 1.0
    d, act, W, X = dev(d), dev(act), dev(rng.standard_normal((out, in_)).astype(np.float32)), dev(rng.standard_normal((B, in_)).astype(np.float32))
    codes, st = torch.full((B, out), 99, dtype=torch.int8, device=DEV), torch.full((32,), 0xEE, dtype=torch.uint8, device=DEV)
    dX, dW, db = (torch.full(s, -7.0, dtype=torch.float32, device=DEV) for s in ((B, in_), (out, in_), (out,)))
    pair, ref_pair = torch.empty(2, dtype=torch.float32, device=DEV), torch.empty(2, dtype=torch.float32, device=DEV)
    ws = torch.empty(dbp.linear_layer_workspace_bytes(B, in_, out), dtype=torch.uint8, device=DEV)
    dbp.dithered_linear_layer_backward(d, act, W, X, dbp.F32, B, in_, out, 3.0, 7, 5, codes, dX, dW, db, pair, ws, st, dbp.PATH_AUTO, stream())
    dbp.step_size(d, act, B * out, 3.0, ref_pair, torch.empty(dbp.step_size_workspace_bytes(B * out), dtype=torch.uint8, device=DEV), stream())
    ref_codes, ref_st = torch.empty_like(codes), torch.zeros_like(st)
    fmt = torch.empty(dbp.format_layout(B, out)["total_bytes"], dtype=torch.uint8, device=DEV)
    dbp.nsd_quantize_ex(d, B, out, 1.0, 7, 5, ref_codes, fmt, ref_st, act=act, step_dev=ref_pair, stream=stream())
    torch.cuda.synchronize()
    assert torch.equal(pair, ref_pair) and torch.equal(codes, ref_codes) and torch.equal(st, ref_st)
    assert (float(pair[0]) > 0.0) == masked and bool(codes.any()) == masked
    assert dbp.Stats.from_tensor(st).n_nonfinite == (0 if masked else 1)
    if not masked:
        assert not pair.any() and not dX.any() and not dW.any() and not db.any()


@pytest.mark.parametrize("what,over", [("dX", "delta"), ("dX", "act"), ("dW", "delta"), ("dW", "act"), ("db", "delta"), ("db", "act"), ("stats", "delta"), ("stats", "act")])
def test_layer_results_in_the_place_of_gradients_or_activations(what, over):
    import paper_2004_04729_amd as dbp
    from gpu_util import DEV, dev, stream
    rng = np.random.default_rng(4)
    n = 64
    d, act = rng.laplace(0, 1e-3, (n, n)).astype(np.float32), rng.standard_normal((n, n)).astype(np.float32)
    W, X = dev(rng.standard_normal((n, n)).astype(np.float32)), dev(rng.standard_normal((n, n)).astype(np.float32))
    ws = torch.empty(dbp.linear_layer_workspace_bytes(n, n, n), dtype=torch.uint8, device=DEV)
    out = []
    for place in (False, True):
        t = {"delta": dev(d), "act": dev(act)}
        r = {"dX": torch.empty((n, n), device=DEV), "dW": torch.empty((n, n), device=DEV), "db": torch.empty(n, device=DEV), "stats": torch.empty(8, device=DEV)}
        if place:
            r[what] = t[over].view(-1)[:r[what].numel()].view(r[what].shape)
        codes, pair = torch.empty((n, n), dtype=torch.int8, device=DEV), torch.empty(2, device=DEV)
        dbp.dithered_linear_layer_backward(t["delta"], t["act"], W, X, dbp.F32, n, n, n, 3.0, 3, 0, codes, r["dX"], r["dW"], r["db"], pair, ws, r["stats"], dbp.PATH_AUTO,
                                           stream())
        torch.cuda.synchronize()
        out.append((codes, pair, r["dX"], r["dW"], r["db"], r["stats"].view(torch.uint8)))
    assert all(torch.equal(a, b) for a, b in zip(*out))
