"""The BF16 network's kernels at the edges of their tiles: widths that fill a
wavefront's tiles and that do not, batches around 16, 64 and the line past
which the weight sum is formed ahead, inputs of one column and of all 64.

Reference: the same network in FP64 with every operand (inputs, weights,
activations, gradients with respect to pre-activations) rounded to BF16 where
the kernels round it, so what is left is FP32 accumulation and the operands
it moves across a rounding boundary: a share of some 1e-4 of them, each by
2^-8, which is 1e-4 normwise in a layer and below 1e-3 through the net."""
import numpy as np
import pytest

from oracle import mlp as omlp

pytestmark = pytest.mark.gpu


def bf16(x):
    u = np.ascontiguousarray(x, np.float32).view(np.uint32).astype(np.uint64)
    u = (u + 0x7fff + ((u >> 16) & 1)) & 0xffff0000
    return u.astype(np.uint32).view(np.float32).astype(np.float64)


def reference(p, X, t, w, n_in, width, skip):
    (W1, b1), (W2, b2), (W3, b3), (W4, b4) = omlp.unpack(p, n_in, width)
    R = [bf16(W) for W in (W1, W2, W3, W4)]
    H, Z = [bf16(X)], []
    for W, b in zip(R[:3], (b1, b2, b3)):
        Z.append(H[-1] @ W.T + b)
        H.append(bf16(omlp.silu(Z[-1])))
    y = H[3] @ R[3][0] + b4[0] + skip[1] * X[:, skip[0]]
    dy = 2.0 * w * (y - t) / w.sum()
    grads = [None] * 4
    grads[3] = (dy[None, :] @ H[3], np.array([dy.sum()]))
    dH = dy[:, None] * R[3]
    for l in (2, 1, 0):
        dZ = dH * omlp.dsilu(Z[l])
        grads[l] = (bf16(dZ).T @ H[l], dZ.sum(axis=0))
        dH = bf16(dZ) @ R[l]
    return y, float((w * (y - t) ** 2).sum() / w.sum()), grads


@pytest.mark.parametrize("n_in,width,B", [(1, 64, 1), (21, 128, 15), (64, 192, 17), (21, 256, 63), (18, 256, 512),
                                          (33, 320, 65), (21, 512, 130), (64, 1024, 48), (21, 256, 4100)])
def test_forward_and_gradient(n_in, width, B):
    import paper_1708_07045_amd as fd
    rng = np.random.default_rng(width + B)
    p = omlp.init_params(n_in, width, rng).astype(np.float32).astype(np.float64)
    N = B + 37
    X = rng.normal(size=(N, n_in)).astype(np.float32).astype(np.float64)
    t = rng.normal(size=N).astype(np.float32).astype(np.float64)
    w = rng.uniform(0.5, 2.0, N).astype(np.float32).astype(np.float64)
    idx = rng.permutation(N)[:B].astype(np.int32)
    skip = (n_in - 1, 0.5)
    net = fd.Network(n_in, width, B)
    net.set_skip(*skip)
    net.set_params(p)
    close = lambda a, b: np.linalg.norm(a - b) <= 1e-3 * np.linalg.norm(b) + 1e-9  # noqa: E731
    y = net.forward(X).cpu().numpy().astype(np.float64)  # more rows than a batch holds
    assert close(y, reference(p, X, t, w, n_in, width, skip)[0])
    loss, g = net.grad(X, t, w, idx)
    yr, lr, gr = reference(p, X[idx], t[idx], w[idx], n_in, width, skip)
    assert loss == pytest.approx(lr, rel=1e-3)
    g = g.cpu().numpy().astype(np.float64)
    for (W, b), (Wr, br) in zip(omlp.unpack(g, n_in, width), gr):
        assert close(W, Wr) and close(b, br)


@pytest.mark.parametrize("rows", [1, 31, 8191, 8192, 8205])
def test_forward_tiles(rows):
    """One and two 16-row tiles a block give the same outputs."""
    import torch
    import paper_1708_07045_amd as fd
    rng = np.random.default_rng(rows)
    net = fd.Network(21, 256, 512)
    net.set_params(omlp.init_params(21, 256, rng))
    X = torch.as_tensor(rng.normal(size=(rows, 21)).astype(np.float32), device="cuda")
    y = net.forward(X)
    parts = torch.cat([net.forward(X[a:a + 1000]) for a in range(0, rows, 1000)])
    assert torch.equal(y, parts)
