"""GPU: infinities stay where the arithmetic puts them.  Sizes are padded inside the kernels; what is padding must not
turn an infinite value into NaN in entries it has no part in."""
import numpy as np
import pytest

from util import to_gpu, to_np

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def bp():
    import torch
    assert torch.cuda.is_available()
    import paper_1907_10134_amd as lib
    return lib


@pytest.mark.parametrize("T,B,H", [(300, 3, 33), (300, 3, 64), (300, 2, 40), (420, 2, 100), (500, 1, 5), (700, 2, 17), (260, 2, 127)])
def test_scan_overflows_to_infinity(bp, T, B, H):
    """Positive Jacobians that grow the gradient 1e17-fold per step, so that segments of a few steps overflow too: no
    bracketing of the products has a 0 * Inf or an Inf - Inf in it, and every gradient is the fp64 chain's, infinite
    where that is beyond fp32."""
    rng = np.random.default_rng(T + H)
    Jt = (rng.uniform(0.5, 1.0, (T, B, H, H)) * (1e17 / (0.75 * H))).astype(np.float32)
    seed = rng.uniform(0.5, 1.0, (B, H)).astype(np.float32)
    got = to_np(bp.scan(to_gpu(Jt), to_gpu(seed))).astype(np.float64)
    assert not np.isnan(got).any(), np.argwhere(np.isnan(got))[:3]
    v, top, seen = seed.astype(np.float64), float(np.finfo(np.float32).max), 0
    for t in range(T - 1, 0, -1):
        v = np.einsum("bij,bj->bi", Jt[t].astype(np.float64), v)
        if v.max() < 1e-3 * top:
            assert np.all(np.abs(got[t - 1] - v) <= 1e-4 * v.max())
            seen += 1
        elif v.min() > 1e3 * top:
            assert np.all(got[:t] == np.inf)
            break
    assert seen == 2


def _with_and_without_infinity(H, I, where, run):
    """run(weights) for a reset gate with a weight of 1e6 and of Inf: its values are 0 or 1 either way."""
    rng = np.random.default_rng(H + I)
    w = {"w_ih": rng.standard_normal((3 * H, I)).astype(np.float32) * 0.2,
         "w_hh": rng.standard_normal((3 * H, H)).astype(np.float32) * 0.2,
         "b_ih": rng.standard_normal(3 * H).astype(np.float32), "b_hh": rng.standard_normal(3 * H).astype(np.float32)}
    T, B = 3, 7
    h = rng.uniform(0.25, 0.75, (T + 1, B, H)).astype(np.float32)
    x = rng.uniform(0.5, 1.0, (T, B, I)).astype(np.float32)
    G = rng.standard_normal((T, B, H)).astype(np.float32)
    out = []
    for value in (1e6, np.inf):
        w[where][5, 0] = value
        out.append(run(to_gpu(h), to_gpu(x), to_gpu(G), [to_gpu(w[k]) for k in ("w_ih", "w_hh", "b_ih", "b_hh")]))
    for finite, infinite in zip(*out):
        assert np.isfinite(finite).all() and np.array_equal(infinite, finite)


GATES = [(20, 3, "w_hh"), (33, 3, "w_hh"), (20, 3, "w_ih"), (33, 17, "w_ih"), (128, 3, "w_ih")]


@pytest.mark.parametrize("H,I,where", GATES)
def test_jacobians_with_an_infinite_gate_weight(bp, H, I, where):
    """Only the entry that multiplies the weight itself, with 0, may differ."""
    def run(h, x, G, w):
        Jt = to_np(bp.build_jacobians(bp.GRU, h, x, *w))
        if where == "w_hh":
            Jt[:, :, 0, 5] = 0.0
        return [Jt] + ([to_np(bp.gru_scan_fused(h, x, *w, G[0].contiguous()))[:2]] if H == 128 else [])

    _with_and_without_infinity(H, I, where, run)


@pytest.mark.parametrize("H,I,where", GATES)
def test_gradients_with_an_infinite_gate_weight(bp, H, I, where):
    _with_and_without_infinity(H, I, where, lambda h, x, G, w: [to_np(g) for g in bp.param_grads(bp.GRU, h, x, G, *w)])
