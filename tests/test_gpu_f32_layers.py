"""fp32 model layers (bf16 matrix cores on exactly split operands) through
rb_run_group, against fp64: every tile shape and its ragged edges, rows read
from the request arena at any alignment, and infinite, NaN and huge values."""
import time

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_1712_06139_amd import rb

pytestmark = pytest.mark.gpu
DEV = "cuda"


@pytest.fixture(scope="module")
def ctx():
    c = rb.Ctx(0)
    yield c
    c.destroy()


def _layers(rng, dims):
    ls = []
    for i, (fi, fo) in enumerate(zip(dims[:-1], dims[1:])):
        W = (rng.standard_normal((fo, fi)) / np.sqrt(fi)).astype(np.float32)
        ls.append((W, rng.uniform(-0.5, 0.5, fo).astype(np.float32), "relu" if i + 2 < len(dims) else "none"))
    return ls


def _run(ctx, layers, X, shift=0, dense_len=None, pad=0.0, allowed=(), poison=False):
    """One group of single-row-block requests (64 rows each, batches of up to
    4096 rows); `shift`: floats before the first row in the arena (NaN with
    `poison`, as are as many after each request)."""
    M, d_in = X.shape
    d_out = layers[-1][0].shape[0]
    m = rb.Model(ctx, "mlp", "f32", layers)
    s = rb.Sched(ctx, pad_value=pad)
    q = rb.Queue(s, m, 4096, allowed)
    first = np.arange(0, M, 64)
    kr = np.zeros(len(first), rb.K_REQ_DTYPE)
    kr["n_rows"] = np.minimum(64, M - first)
    gap = shift if poison else 0
    kr["dense_off"] = shift + first * d_in + np.arange(len(first)) * gap
    kr["dense_end"] = kr["dense_off"] + kr["n_rows"] * d_in
    kr["out_off"] = first * d_out
    nb = (M + 4095) // 4096
    kb = np.zeros(nb, rb.K_BATCH_DTYPE)
    for b in range(nb):
        real = min(4096, M - b * 4096)
        kb[b] = (b * 64, (real + 63) // 64, b * 4096, min([a for a in allowed if a >= real], default=real), real, 0)
    slots = int(kb["row_base"][-1] + kb["padded"][-1])
    dense = torch.full((shift + M * d_in + len(first) * gap,), float("nan") if poison else 0.0, device=DEV)
    out = torch.full((M * d_out,), -7.0, device=DEV)
    up = [torch.from_numpy(a.view(np.uint8)).to(DEV) for a in (kb, kr)]
    for o, e, r in zip(kr["dense_off"], kr["dense_end"], first):
        dense[o:e] = torch.from_numpy(X[r:r + 64].reshape(-1)).to(DEV)
    torch.cuda.synchronize()
    q.run_group(0, up[0], nb, up[1], len(kr), slots, 0, dense, dense.numel() if dense_len is None else dense_len, None,
                0, None, 0, out, out.numel())
    status = rb.lib().rb_sync(s.h)
    y = out.cpu().numpy().reshape(M, d_out)
    q.destroy()
    s.destroy()
    m.destroy()
    return y, status


def _ref(layers, X):
    x = X.astype(np.float64)
    with np.errstate(all="ignore"):
        for i, (W, b, act) in enumerate(layers):
            x = x @ W.astype(np.float64).T + b
            x = (np.where(x > 0, x, 0) if act == "relu" else x).astype(np.float32).astype(np.float64)
    return x


def _err(y, ref):
    return np.max(np.abs(y - ref) / np.maximum(np.abs(ref).max(axis=1, keepdims=True), 1e-30))


# rows around the 32- and 64-row tiles; widths for each tile (N a multiple
# of 64, 128, 256); 33000 rows x 512 and 66000 x 256 take the 64 x 256 tile on
# 256 compute units, 8256 x 256 the 64 x 128 one. d_in not a multiple of 64 is
# assembled first, the others are read from the arena, aligned or not.
@pytest.mark.parametrize("M,dims,shift", [
    (1, (64, 128, 16), 0), (31, (64, 64), 1), (33, (128, 40, 3), 2), (65, (100, 300, 70), 3), (127, (256, 1024, 32), 0),
    (129, (320, 192), 1), (8256, (64, 256, 128), 3), (33000, (64, 512, 256), 1), (66000, (128, 256), 0)])
def test_f32_layers_match_fp64(ctx, M, dims, shift):
    rng = np.random.default_rng(M)
    layers, X = _layers(rng, dims), rng.standard_normal((M, dims[0])).astype(np.float32)
    y, status = _run(ctx, layers, X, shift)
    assert status == rb.RB_OK
    # over all outputs: one rounding for 8 of up to 1024 products, 2e-7 of the norm
    # at most (measured 1.8e-7), over two layers; without one of the smaller partial
    # products it would be 2e-6 and more
    ref = _ref(layers, X)
    assert np.linalg.norm(y - ref) <= 4e-7 * np.linalg.norm(ref)
    assert _err(y, ref) <= 1e-5
    # a row's bits do not depend on the rows it runs with, nor on its alignment
    for r0, n in ((0, 1), (M // 2, min(40, M - M // 2)), (M - 1, 1)):
        part, _ = _run(ctx, layers, X[r0:r0 + n], (shift + 1) % 4)
        assert np.array_equal(part, y[r0:r0 + n])


def test_f32_layer_exact_products(ctx):
    # one-hot rows return weights exactly: no bits of an operand are lost
    W = np.random.default_rng(1).standard_normal((64, 64)).astype(np.float32)
    W[:, 5] *= np.float32(1e-30)
    W[:, 6] *= np.float32(1e30)
    y, _ = _run(ctx, [(W, np.zeros(64, np.float32), "none")], np.eye(64, dtype=np.float32))
    assert np.array_equal(y, W.T)


# the 32 x 64, 64 x 128 and 64 x 256 tiles
@pytest.mark.parametrize("M,N,K", [(256, 64, 64), (512, 256, 1024), (8256, 256, 256), (66000, 256, 192)])
@pytest.mark.parametrize("density", [1.0, 0.5, 0.1, 0.02])
def test_f32_layer_error_is_no_larger_than_the_fp32_mfma_kernels(ctx, M, N, K, density):
    # dense inputs, inputs half zeros (a hidden layer's after a ReLU) and sparse
    # ones: the error against 64 bits, over all outputs, is at most that of the
    # kernel on fp32 operands (its sums have no fewer roundings)
    rng = np.random.default_rng(K + N)
    W = (rng.standard_normal((N, K)) / np.sqrt(K)).astype(np.float32)
    b = np.zeros(N, np.float32)
    X = (rng.standard_normal((M, K)) * (rng.random((M, K)) < density)).astype(np.float32)
    y, _ = _run(ctx, [(W, b, "none")], X)
    Xd, Wd, bd = (torch.from_numpy(a).to(DEV) for a in (X, W, b))
    Y = torch.empty(M, N, device=DEV)
    rb.check(rb.lib().rb_k_gemm_f32(rb.torch_stream_ptr(), rb.dptr(Xd), K, rb.dptr(Wd), K, rb.dptr(bd), rb.dptr(Y), N,
                                    M, N, K, rb.RB_ACT_NONE, None, 0), "rb_k_gemm_f32")
    ref = Xd.double() @ Wd.double().T
    err = [float((torch.as_tensor(v).to(DEV).double() - ref).norm() / ref.norm()) for v in (y, Y)]
    assert err[0] <= err[1], err


@pytest.mark.parametrize("M,K", [(1, 64), (40, 192), (8256, 256), (40000, 512)])
def test_f32_layer_exact_products_of_inputs(ctx, M, K):
    # the identity as weights returns the inputs exactly, on each tile (32 x 64,
    # 64 x 128, 64 x 256) and in every k-step: no bits of X's three parts are lost
    # or misplaced, whatever its scale
    X = np.random.default_rng(K).standard_normal((M, K)).astype(np.float32)
    X[:, 3::7] *= np.float32(1e-38)
    X[:, 5::7] *= np.float32(1e22)
    y, _ = _run(ctx, [(np.eye(K, dtype=np.float32), np.zeros(K, np.float32), "none")], X)
    assert np.array_equal(y, X)


@pytest.mark.parametrize("M,N", [(64, 64), (8256, 256), (66000, 256)])
@pytest.mark.parametrize("e", [100, 109, 110, 111, 115, 126, 135, 148])
def test_f32_layer_keeps_the_bits_of_tiny_values(ctx, M, N, e):
    # values around 2^-110, under which three bf16 parts no longer hold an fp32
    # value, down to the smallest one: as inputs against weights of 1 to 2^120,
    # and as weights. Every product here is an fp32 value, so outputs are exact.
    rng = np.random.default_rng(e)
    bits = min(24, 150 - e)  # of the values' significands
    tiny = lambda n: np.ldexp(rng.integers(1 << (bits - 1), 1 << bits, n).astype(np.float64), 1 - bits - e)  # noqa: E731
    rows = np.unique(np.concatenate([np.arange(0, M, max(1, M // 50)), [M - 1]]))
    k = rng.integers(0, 64, len(rows))
    x = tiny(len(rows)).astype(np.float32)
    b = np.zeros(N, np.float32)
    for s in (0, 60, 120):
        X = rng.standard_normal((M, 64)).astype(np.float32)
        W = np.zeros((N, 64), np.float32)
        W[:, :] = np.ldexp(1.0, s + np.arange(N) % 2)[:, None]
        W[N - 1] = 0.25
        base, _ = _run(ctx, [(W, b, "none")], X)
        X[rows] = 0
        X[rows, k] = x
        y, _ = _run(ctx, [(W, b, "none")], X)
        want = x.astype(np.float64)[:, None] * W[:, 0].astype(np.float64)
        exact = want == want.astype(np.float32)
        assert exact[:, :N - 1].all() and np.array_equal(y[rows][exact], want[exact].astype(np.float32)), s
        other = np.setdiff1d(np.arange(M), rows)
        assert np.array_equal(y[other], base[other])
        # the same values as weights (W of N rows, one value each), inputs 2^s
        W = np.zeros((N, 64), np.float32)
        w, kw = tiny(N).astype(np.float32), rng.integers(0, 64, N)
        W[np.arange(N), kw] = w
        y, _ = _run(ctx, [(W, b, "none")], np.full((M, 64), 2.0 ** s, np.float32))
        assert np.array_equal(y, np.tile((w.astype(np.float64) * 2.0 ** s).astype(np.float32), (M, 1))), s


def test_f32_layer_tiny_values_beside_ordinary_ones(ctx):
    # a tiny value counts where its product does, and nowhere else
    X = np.zeros((40, 64), np.float32)
    X[:, 0] = np.float32(1.2345678) * np.float32(2.0 ** -120)
    X[:, 1] = 1.0
    W = np.zeros((64, 64), np.float32)
    W[0, 0], W[0, 1] = 2.0 ** 120, 1.0   # 1 + 1.2345678
    W[1, 0], W[1, 1] = 1.0, 1.0          # 1 + 2^-120: 1
    W[2, 0], W[2, 1] = 2.0 ** 100, 0.0   # 2^-20
    y, _ = _run(ctx, [(W, np.zeros(64, np.float32), "none")], X)
    x = float(X[0, 0])
    assert np.array_equal(y[:, 0], np.full(40, np.float32(1.0 + x * 2.0 ** 120)))
    assert np.array_equal(y[:, 1], np.ones(40, np.float32))
    assert np.array_equal(y[:, 2], np.full(40, np.float32(x * 2.0 ** 100))) and not y[:, 3:].any()


@pytest.mark.parametrize("N,K", [(1, 1), (33, 17), (70, 100), (64, 64)])
def test_f32_weights_keep_their_bits(ctx, N, K):
    # one-hot inputs return every weight of widths that are padded, exactly: the
    # largest finite ones, subnormal ones beside them in other layers, infinities
    rng = np.random.default_rng(N)
    for scale in (1e-44, 1.0, 3e37):
        W = (rng.standard_normal((N, K)) * scale).astype(np.float32)
        W[0, 0] = np.float32(3.4028235e38) if scale > 1 else np.float32(-0.0)
        y, _ = _run(ctx, [(W, np.zeros(N, np.float32), "none")], np.eye(K, dtype=np.float32))
        assert np.array_equal(y, W.T)
    W[N - 1, K - 1] = -np.inf
    y, _ = _run(ctx, [(W, np.zeros(N, np.float32), "none")], np.eye(K, dtype=np.float32))
    hot = np.ones((K, N), bool)
    hot[:, N - 1] = False  # 0 times infinity
    hot[K - 1, N - 1] = True
    assert np.array_equal(y[hot], W.T[hot]) and np.isnan(y[~hot]).all()


def test_f32_model_loads_about_as_fast_as_it_copies(ctx):
    # a 4096 x 4096 fp32 layer within 4 times a bf16 one's time (measured 1.5;
    # split element by element on the host it was 10)
    W, b = np.random.default_rng(0).standard_normal((4096, 4096)).astype(np.float32), np.zeros(4096, np.float32)
    best = {}
    for dtype in ("bf16", "f32") * 4:
        t0 = time.perf_counter()
        m = rb.Model(ctx, "mlp", dtype, [(W, b, "none")])
        best[dtype] = min(best.get(dtype, 1e9), time.perf_counter() - t0)
        m.destroy()
    assert best["f32"] <= 4 * best["bf16"], best


def test_f32_layers_tiny_weights_and_huge_inputs(ctx):
    # a tiny weight scales its layer: sums that overflow for it (or for X's own
    # scale) are computed on fp32 operands, from the unscaled weights
    rng = np.random.default_rng(7)
    W = (rng.standard_normal((128, 64)) / 8).astype(np.float32)
    W[0, 0] = 1e-44
    X = rng.standard_normal((100, 64)).astype(np.float32)
    X[3], X[5], X[7] = X[3] * np.float32(1e17), X[5] * np.float32(1e30), X[7] * np.float32(1e37)
    X[9] = X[9] * np.float32(1e-36)
    y, _ = _run(ctx, [(W, np.zeros(128, np.float32), "none")], X)
    assert _err(y, X.astype(np.float64) @ W.astype(np.float64).T) <= 1e-6


@pytest.mark.parametrize("M", [40, 33000])
def test_f32_layers_non_finite_and_huge(ctx, M):
    # rows with infinities, NaN and values whose products or bf16 roundings
    # overflow give what fp32 arithmetic gives; their neighbours keep their bits
    rng = np.random.default_rng(3)
    W = np.abs(rng.standard_normal((512, 64))).astype(np.float32)
    W[7, 3] = np.float32(3.4e38)
    W[9, 2] = np.inf
    layers = [(W, np.zeros(512, np.float32), "none")]
    X = np.abs(rng.standard_normal((M, 64))).astype(np.float32)
    X[:, 2:4] = np.float32(0.25)
    base, _ = _run(ctx, layers, X)
    X2 = X.copy()
    X2[3, 10], X2[5, 11], X2[9, 12], X2[11, 0] = np.inf, np.nan, np.float32(3.4e38), np.float32(-np.inf)
    X2[13, :] = np.float32(1e38)
    y, _ = _run(ctx, layers, X2)
    same = np.setdiff1d(np.arange(M), [3, 5, 9, 11, 13])
    assert np.array_equal(y[same], base[same], equal_nan=True)
    with np.errstate(all="ignore"):
        ref = X2[:16].astype(np.float64) @ W.astype(np.float64).T
        ref32 = ref.astype(np.float32)
    fin = np.isfinite(ref32) & (np.abs(ref) < 1e38)
    assert np.max(np.abs(y[:16][fin] - ref[fin]) / np.abs(ref[fin])) <= 1e-5
    assert np.array_equal(np.isnan(y[:16]), np.isnan(ref32))
    big = np.abs(ref) > 1e39
    assert np.array_equal(y[:16][big], ref32[big])


def test_f32_layers_rows_outside_the_arena(ctx):
    # the last request's rows end past the declared arena: reported, and they
    # contribute zeros; other rows are unchanged. NaN padding (rows assembled) and
    # NaN around and between the requests' rows (read in place) reach nothing.
    rng = np.random.default_rng(5)
    layers, X = _layers(rng, (64, 128, 16)), rng.standard_normal((150, 64)).astype(np.float32)
    good, status = _run(ctx, layers, X, pad=float("nan"), allowed=(256, 4096))
    assert status == rb.RB_OK and np.isfinite(good).all()
    inplace, status = _run(ctx, layers, X, shift=5, allowed=(256, 4096), poison=True)
    assert status == rb.RB_OK and np.array_equal(inplace, good)
    y, status = _run(ctx, layers, X, dense_len=149 * 64 + 10)
    assert status == rb.RB_ERANGE
    assert np.array_equal(y[:149], good[:149])
    assert _err(y[149:], _ref(layers, np.zeros((1, 64), np.float32))) <= 1e-5
