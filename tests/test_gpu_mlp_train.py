"""The fused training step of the learned warm start (padded layer widths up to 256) over its
tilings: ragged row counts, narrow and full layers, no hidden layer up to four, both dtypes,
and the weight copies the optimiser step keeps (checked bit for bit against a fresh handle
given the same parameters).

Gradients are compared with the FP64 reference's layers evaluated with BF16 rounding at the
kernel's own rounding points (features, weights, every activation and every back-propagated
gradient).  What is left are FP32 sums and exponentials, 2^-20 or so relative, which now and
then (one entry in 2^12) tip a BF16 rounding of 2^-8: in the norm of a layer's gradient
2^-14 per rounding point, so (L + 1) 2^-10 leaves a factor of ten; where a layer has too few
entries for that (below 2,000) every one of its 2 L + 2 rounding points may tip.
"""
import numpy as np
import pytest
import torch

from oracle import mlp_ref as M
import paper_2403_04578_amd as tpf
from paper_2403_04578_amd import workloads as W
from test_gpu_mlp import _ref_params, bf16_round

pytestmark = pytest.mark.gpu


def _batch(gpu, n, rows, dtype):
    f = W.make_feeder(n + 1)
    S = torch.from_numpy(W.profile_minute_year(f, steps=rows, seed=n)).to(dtype)
    rng = np.random.default_rng(rows)
    V = torch.from_numpy(1.0 + 0.05 * (rng.standard_normal((rows, n)) + 1j * rng.standard_normal((rows, n)))).to(dtype)
    t = np.arange(rows, dtype=np.int64) * 977 % W.MINUTES_PER_YEAR
    return S.to(gpu), torch.from_numpy(t).to(gpu), V.to(gpu), S.numpy().astype(np.complex128), t, V.numpy().astype(np.complex128)


def _rounded_reference(p0, sizes, S, t, V):
    """(loss, flat gradient) with BF16 rounding where the kernel rounds."""
    layers = M.unpack(_ref_params(p0, sizes), sizes)
    f32 = np.float32(50.0) * np.concatenate([S.real, S.imag], axis=1).astype(np.float32)
    h = [np.concatenate([bf16_round(f32), bf16_round(M.features(S, t)[:, -4:])], axis=1)]
    z = []
    for W_, b in layers[:-1]:
        z.append(h[-1] @ W_.T + b)
        h.append(bf16_round(M.gelu(z[-1])))
    y = h[-1] @ layers[-1][0].T + layers[-1][1]
    d = y - M.targets(V)
    out, dz = [], bf16_round(2.0 / d.size * d)
    for l in range(len(layers) - 1, -1, -1):
        out = [(dz.T @ h[l]).ravel(), dz.sum(0)] + out
        if l:
            dz = bf16_round((dz @ layers[l][0]) * M.gelu_grad(z[l - 1]))
    return float((d * d).mean()), np.concatenate(out)


@pytest.mark.parametrize("n,hidden,layers,rows,dtype", [
    (1, 1, 1, 1, torch.complex128), (5, 17, 2, 7, torch.complex64), (30, 64, 0, 9, torch.complex128),
    (31, 65, 1, 64, torch.complex64), (62, 128, 4, 65, torch.complex128), (99, 256, 3, 8, torch.complex128),
    (99, 200, 2, 257, torch.complex64), (126, 256, 3, 300, torch.complex128)])
def test_gradient_at_every_tiling(gpu, n, hidden, layers, rows, dtype):
    Sd, td, Vd, S, t, V = _batch(gpu, n, rows, dtype)
    sizes = W.mlp_sizes(n, hidden, layers)
    p0 = W.mlp_init_params(sizes, seed=n + layers)
    loss, grad = tpf.WarmStart(n, hidden, layers, p0).loss_grad(Sd, td, Vd)
    g = grad.cpu().numpy().astype(np.float64)
    lref, gref = _rounded_reference(p0, sizes, S, t, V)
    assert abs(float(loss) - lref) <= 1e-3 * lref
    bound = (layers + 1) * 2.0 ** -10 if rows * hidden >= 2000 else (2 * layers + 2) * 2.0 ** -8
    o = 0
    for a, b in zip(sizes[:-1], sizes[1:]):
        for count in (a * b, b):
            e = np.linalg.norm(g[o:o + count] - gref[o:o + count])
            assert e <= bound * np.linalg.norm(gref[o:o + count]) + 1e-12, (a, b, count)
            o += count


@pytest.mark.parametrize("n,hidden,layers", [(7, 40, 2), (99, 256, 3), (126, 256, 1), (140, 256, 2), (60, 300, 1)])
def test_optimiser_step_keeps_the_weight_copies(gpu, n, hidden, layers):
    """After an epoch of training the handle predicts and differentiates exactly as a new one
    built from its parameters (the last two sizes take the per-layer kernels)."""
    Sd, td, Vd, *_ = _batch(gpu, n, 200, torch.complex128)
    a = tpf.WarmStart(n, hidden, layers, W.mlp_init_params(W.mlp_sizes(n, hidden, layers), seed=3))
    losses = a.fit(Sd, td, Vd, epochs=2, batch=48, lr=1e-3, seed=5)
    assert len(losses) == 2 and all(np.isfinite(losses)) and losses[1] < losses[0]
    b = tpf.WarmStart(n, hidden, layers, a.get_params())
    assert torch.equal(a.predict(Sd, td), b.predict(Sd, td))
    ga, gb = a.loss_grad(Sd, td, Vd)[1], b.loss_grad(Sd, td, Vd)[1]
    assert torch.equal(ga, gb)
