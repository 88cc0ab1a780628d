"""Matrix products of the learned proposal at the edges of their tiles: batches,
widths and sequence lengths that are no multiples of 16 or 32, wave tiles of
both sizes, and a smaller batch after a larger one (rows left over from the
larger batch must not enter the sums over the batch).

Tolerances: a product of bf16 operands accumulated in fp32 differs from the
double-precision sum by at most 2 K 2^-24 sum |a b|; column sums of K fp32
terms likewise; the epilogue multiplications add a few ulp.  K counts whole
steps of 32, as the instruction sums them."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _bound(A, B):
    return 2.0 * ((A.shape[1] + 31) // 32 * 32) * 2.0 ** -24 * (np.abs(A) @ np.abs(B))


@pytest.mark.parametrize("M,T,nu,H", [
    (1, 1, 2, 1), (7, 5, 3, 17), (31, 9, 2, 33), (33, 20, 3, 48), (300, 40, 2, 250), (2047, 21, 3, 130), (8100, 20, 2, 290),
])
def test_products_at_tile_edges(M, T, nu, H):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2605_29663_amd as pkg
    from oracle import mlp
    net = pkg.Proposal(T, nu, hidden=H, max_batch=M + 40)
    In, O = net.in_dim, net.out_dim
    rng = np.random.default_rng(M)
    theta = mlp.pack(*(rng.normal(0, 0.2, s) for s in ((In, H), H, (H, H), H, (H, O), O))).astype(np.float32)
    net.set_params(theta)
    big = M + 40
    Xb, Yb = (torch.tensor(rng.uniform(-1, 1, (big, c)).astype(np.float32), device="cuda") for c in (In, O))
    net.train_step(Xb, Yb, lr=0.0)
    X, Y = rng.uniform(-1, 1, (M, In)).astype(np.float32), rng.uniform(-1, 1, (M, O)).astype(np.float32)
    Xd, Yd = torch.tensor(X, device="cuda"), torch.tensor(Y, device="cuda")
    loss = net.train_step(Xd, Yd, lr=0.0)
    g = lambda name, cols: net.get_buffer(name, M * cols).astype(np.float64).reshape(M, cols)
    x, a1, a2 = g("x", In), g("a1", H), g("a2", H)
    pre1, pre2, out = g("pre1", H), g("pre2", H), g("out", O)
    dout, dout_b, dh2, dh2_b, dh1, dh1_b = (g(*v) for v in (("dout", O), ("dout_b", O), ("dh2", H), ("dh2_b", H),
                                                            ("dh1", H), ("dh1_b", H)))
    W1, b1, W2, b2, W3, b3 = mlp.unpack(theta.astype(np.float64), In, H, O)
    np.testing.assert_array_equal(x, mlp.bf16(X))
    for A, W, b, y in ((x, W1, b1, pre1), (a1, W2, b2, pre2), (a2, W3, b3, out)):
        Wb = mlp.bf16(W)
        assert np.all(np.abs(y - (A @ Wb + b)) <= _bound(A, Wb) + 1e-6 * np.abs(y) + 1e-7)
    for b16, f32 in ((dout_b, dout), (dh2_b, dh2), (dh1_b, dh1)):
        np.testing.assert_array_equal(b16, mlp.bf16(f32))
    np.testing.assert_allclose(dout, 2.0 * (out - Y) / (M * O), rtol=1e-6, atol=1e-7 / (M * O))
    np.testing.assert_allclose(loss, np.mean((out - Y) ** 2), rtol=1e-5)
    for dY, W, pre, dh in ((dout_b, W3, pre2, dh2), (dh2_b, W2, pre1, dh1)):
        Wb, gg = mlp.bf16(W).T, mlp.gelu_grad(pre)
        ref = (dY @ Wb) * gg
        tol = _bound(dY, Wb) * (np.abs(gg) + 1e-5) + 1e-6 * np.abs(dY @ Wb) + 1e-12
        assert np.all(np.abs(dh - ref) <= tol)
    gW1, gb1, gW2, gb2, gW3, gb3 = mlp.unpack(net.get_buffer("grad", net.n_params).astype(np.float64), In, H, O)
    for A, dY, gW in ((a2, dout_b, gW3), (a1, dh2_b, gW2), (x, dh1_b, gW1)):
        assert np.all(np.abs(gW - A.T @ dY) <= _bound(A.T, dY) + 1e-12)
    for d, gb in ((dout, gb3), (dh2, gb2), (dh1, gb1)):
        assert np.all(np.abs(gb - d.sum(0)) <= 2.0 * M * 2.0 ** -24 * np.abs(d).sum(0) + 1e-12)
    # inference after training leaves the same outputs
    np.testing.assert_array_equal(net.forward(Xd).cpu().numpy(), out.astype(np.float32))
