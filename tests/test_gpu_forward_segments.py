"""GPU: bppsa_forward where it walks a long sequence as segments at the same time.  Whatever the weights, the states
are those of the walk from the start: compared with the same call on pieces too short to be cut, and with the oracle."""
import numpy as np
import pytest

import workloads
from oracle import gru as ogru
from oracle import rnn as orn
from util import to_gpu, to_np

pytestmark = pytest.mark.gpu

PIECE = 96           # no sequence below 120 steps is cut; even, as the wave form alternates between even and odd steps


@pytest.fixture(scope="module")
def bp():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_1907_10134_amd as lib
    return lib


def _inputs(cell, T, B, H, I, gain, seed=0):
    rng = np.random.default_rng(seed + T + H)
    w = workloads.rnn_inputs(T, B, H, I, 10, seed=T + H) if cell == "rnn" else workloads.gru_inputs(T, B, H, I, 11, seed=T + H)
    if cell == "rnn":
        w["b_ih"], w["b_hh"] = w["b"], None
    w["w_hh"] = (gain * w["w_hh"]).astype(np.float32)
    return w, (0.3 * rng.standard_normal((B, H))).astype(np.float32)


def _run(bp, cell, w, h0, piece=None):
    import torch
    T, B, _ = w["x"].shape
    h = torch.full((T + 1,) + h0.shape, 7.0, dtype=torch.float32, device="cuda")
    h[0] = to_gpu(h0)
    x = to_gpu(w["x"])
    weights = [None if w[k] is None else to_gpu(w[k]) for k in ("w_ih", "w_hh", "b_ih", "b_hh")]
    code = bp.RNN_TANH if cell == "rnn" else bp.GRU
    step = piece or T
    for t in range(0, T, step):
        n = min(step, T - t)
        bp.forward(code, x[t:t + n], *weights, h[t:t + n + 1])
    return to_np(h)


def _oracle(cell, w, h0):
    if cell == "rnn":
        return orn.forward(w["x"], w["w_ih"], w["w_hh"], w["b"], h0=h0)
    ref = [h0.astype(np.float64)]
    for x in w["x"]:
        ref.append(ogru.step(ref[-1], x, w["w_ih"], w["w_hh"], w["b_ih"], w["b_hh"]))
    return np.asarray(ref)


SIZES = [("rnn", 1000, 16, 20, 1), ("rnn", 337, 3, 20, 1), ("rnn", 1009, 5, 20, 4), ("rnn", 513, 2, 5, 1), ("rnn", 600, 3, 8, 3),
         ("rnn", 301, 7, 9, 1), ("rnn", 272, 1, 21, 1), ("rnn", 499, 2, 32, 2), ("rnn", 999, 700, 20, 1), ("rnn", 300, 7, 64, 1),
         ("rnn", 351, 2, 33, 5), ("rnn", 288, 1, 128, 40), ("rnn", 400, 2, 20, 5), ("gru", 517, 4, 20, 24), ("gru", 333, 3, 8, 12),
         ("gru", 260, 2, 33, 2), ("gru", 700, 1, 97, 33), ("gru", 250, 5, 128, 1), ("gru", 300, 1, 64, 13)]


@pytest.mark.parametrize("cell,T,B,H,I", SIZES)
def test_segments_match_the_oracle(bp, cell, T, B, H, I):
    w, h0 = _inputs(cell, T, B, H, I, 1.0)
    got, ref = _run(bp, cell, w, h0), _oracle(cell, w, h0)
    assert np.max(np.abs(got - ref)) <= 2e-6          # as for sequences walked in one go
    assert np.max(np.abs(got - _run(bp, cell, w, h0, PIECE))) <= 2e-6


@pytest.mark.parametrize("cell,T,B,H,I", [s for s in SIZES if s[2] < 100])
def test_segments_of_cells_that_amplify(bp, cell, T, B, H, I):
    """Chaotic weights: a wrong start would show at the size of the states, which are O(1), at the next seam at the
    latest.  Seams that do not hold are walked again, so what is left is the walk from the start."""
    w, h0 = _inputs(cell, T, B, H, I, 12.0)
    assert np.max(np.abs(_run(bp, cell, w, h0) - _run(bp, cell, w, h0, PIECE))) <= 2e-6


@pytest.mark.parametrize("gain", [2.0, 3.0])
@pytest.mark.parametrize("cell,T,B,H,I", [s for s in SIZES if s[2] < 100])
def test_segments_of_cells_that_forget_slowly(bp, cell, T, B, H, I, gain):
    """Some seams hold, some do not, and what a seam leaves (a rounding of its step) may grow as the rounding of
    every step does: the states are about as far from the oracle's as those of the walk from the start."""
    w, h0 = _inputs(cell, T, B, H, I, gain)
    ref = _oracle(cell, w, h0)
    off, base = (np.linalg.norm(_run(bp, cell, w, h0, p) - ref) for p in (None, PIECE))
    assert off <= 2 * base + 1e-7 * np.linalg.norm(ref)


@pytest.mark.parametrize("T,B", [(700, 3), (1500, 16)])
def test_segments_with_a_norm_preserving_recurrence(bp, T, B):
    """No seam holds: the bits of the walk from the start."""
    w = workloads.rnn_inputs_norm_preserving(T, B, seed=T)
    w["b_ih"], w["b_hh"] = w["b"], None
    h0 = np.zeros((B, 20), np.float32)
    assert np.array_equal(_run(bp, "rnn", w, h0), _run(bp, "rnn", w, h0, PIECE))


@pytest.mark.parametrize("cell,T,B,H,I", [("rnn", 600, 4, 20, 1), ("rnn", 400, 4, 64, 1), ("gru", 517, 4, 20, 24)])
def test_a_nan_in_one_sample_goes_on_to_its_end_and_nowhere_else(bp, cell, T, B, H, I):
    w, h0 = _inputs(cell, T, B, H, I, 1.0)
    clean = _run(bp, cell, w, h0)
    w["x"] = w["x"].copy()
    w["x"][T // 3, 1, 0] = np.nan
    got = _run(bp, cell, w, h0)
    assert np.isnan(got[T // 3 + 1:, 1]).all()
    assert np.array_equal(got[:T // 3 + 1, 1], clean[:T // 3 + 1, 1])
    assert np.array_equal(np.delete(got, 1, axis=1), np.delete(clean, 1, axis=1))


@pytest.mark.parametrize("gain", [1.0, 12.0])
@pytest.mark.parametrize("T,B,H,I", [(700, 5, 20, 1), (333, 3, 8, 2), (1000, 2, 31, 4)])
def test_training_iteration_on_segments_takes_the_last_state(bp, T, B, H, I, gain):
    """The head of an iteration runs behind the seams: its seed is that of the states as they end up."""
    import torch
    rng = np.random.default_rng(T)
    shapes = bp.binding.rnn_param_shapes(H, I, 10)
    p = {k: torch.from_numpy((rng.uniform(-1, 1, shapes[k]) / np.sqrt(H)).astype(np.float32)).cuda() for k in bp.RNN_PARAM_ORDER}
    p["w_hh"] *= gain
    x = to_gpu(rng.standard_normal((T, B, I)).astype(np.float32))
    labels = to_gpu(rng.integers(0, 10, B).astype(np.int32))
    tr = bp.RnnTrainer(T, B, H, I, 10, {k: v.clone() for k, v in p.items()})
    tr.step(x, labels)
    h = torch.zeros_like(tr.h)
    bp.forward(bp.RNN_TANH, x, p["w_ih"], p["w_hh"], p["b_ih"], p["b_hh"], h)
    assert torch.equal(h, tr.h)
    seed, _ = bp.head_seed(h[T], p["w_out"], p["b_out"], labels)
    assert torch.allclose(tr.seed, seed, rtol=1e-5, atol=1e-8)


# more samples than segments have room for, up to the compute units, and one more than those
ROUNDS = [(288, 100, 20, 1), (289, 65, 20, 1), (290, 256, 5, 2), (385, 130, 8, 4), (1000, 100, 32, 1), (611, 256, 9, 3),
          (400, 257, 20, 1)]


@pytest.mark.parametrize("gain", [1.0, 2.0, 12.0])
@pytest.mark.parametrize("T,B,H,I", ROUNDS)
def test_rounds_of_walks(bp, T, B, H, I, gain):
    w, h0 = _inputs("rnn", T, B, H, I, gain)
    got, pieces = _run(bp, "rnn", w, h0), _run(bp, "rnn", w, h0, PIECE)
    if gain == 2.0:                                   # as above for cells that forget slowly
        ref = _oracle("rnn", w, h0)
        assert np.linalg.norm(got - ref) <= 2 * np.linalg.norm(pieces - ref) + 1e-7 * np.linalg.norm(ref)
    else:
        assert np.max(np.abs(got - pieces)) <= 2e-6


# ---- units of every scale and memory -------------------------------------------------------------------------------
# What a seam may leave is the rounding of a step of that very unit, however large the others are: each unit by itself
# is as near to the oracle as in the walk from the start (twice its error and one rounding of the value).

def _unit_errors(got, ref):
    d, n = got - ref, np.sqrt((ref ** 2).sum(axis=(0, 1)))
    return np.sqrt((d ** 2).sum(axis=(0, 1))) / np.where(n > 0, n, 1)


def _check_units(bp, cell, w, h0):
    ref = _oracle(cell, w, h0)
    got, base = (_unit_errors(_run(bp, cell, w, h0, p), ref) for p in (None, PIECE))
    assert np.all(got <= 2 * base + 2.0 ** -24), (got, base)


def _uncoupled(cell, T, B, H, I, keep):
    """Units that each keep `keep` of their state from step to step, of scales from 1 down to 1e-10, and a last one that
    is always large."""
    rng = np.random.default_rng(T + B + H)
    scale = 10.0 ** -(np.arange(H) % 11)
    x = rng.uniform(0.5, 1.5, (T, B, I)).astype(np.float32)
    if cell == "rnn":
        w_ih, b = np.repeat(0.5 * (1 - keep) / I * scale[:, None] + 1e-9 * scale[:, None], I, axis=1), np.zeros(H)
        w_hh = np.diag(np.full(H, keep))
        w_hh[-1], b[-1] = 0.0, 3.0
        w = dict(w_ih=w_ih, w_hh=w_hh, b_ih=b, b=b)
    else:
        w_ih, b = np.zeros((3 * H, I)), np.zeros(3 * H)
        w_ih[2 * H:] = 0.1 / I * scale[:, None]
        b[H:2 * H], b[2 * H - 1], b[3 * H - 1] = np.log(keep / (1 - keep)), 0.0, 3.0
        w = dict(w_ih=w_ih, w_hh=np.zeros((3 * H, H)), b_ih=b, b_hh=np.zeros(3 * H))
    w = {k: v.astype(np.float32) for k, v in w.items()}
    w.setdefault("b_hh", None)
    return dict(w, x=x), np.zeros((B, H), np.float32)


@pytest.mark.parametrize("gain", [1.0, 1.5, 2.0])
@pytest.mark.parametrize("cell,T,B,H,I", [s for s in SIZES if s[2] < 100] + [("rnn", 1000, 16, 64, 1), ("rnn", 1000, 100, 20, 1)])
def test_units_of_cells_that_forget(bp, cell, T, B, H, I, gain):
    """Where some seams hold by little: recurrent weights 1.5 times as large."""
    _check_units(bp, cell, *_inputs(cell, T, B, H, I, gain))


# segments and rounds of the wave form, block form of both cells
KEEPING = [("rnn", 1000, 16, 20, 1), ("rnn", 9999, 13, 20, 1), ("rnn", 1000, 5, 7, 2), ("rnn", 700, 4, 32, 4),
           ("rnn", 1000, 100, 20, 1), ("rnn", 600, 256, 9, 3), ("rnn", 1000, 4, 64, 1), ("rnn", 600, 4, 20, 5),
           ("rnn", 700, 1, 128, 40), ("gru", 1000, 4, 20, 1), ("gru", 517, 32, 20, 24), ("gru", 1500, 3, 128, 1),
           ("gru", 700, 5, 61, 13)]


@pytest.mark.parametrize("keep", [0.5, 0.8, 0.86, 0.9, 0.95, 0.99, 0.999, 0.99998])
@pytest.mark.parametrize("cell,T,B,H,I", KEEPING)
def test_units_of_every_scale_and_memory(bp, cell, T, B, H, I, keep):
    _check_units(bp, cell, *_uncoupled(cell, T, B, H, I, keep))


@pytest.mark.parametrize("cell,T,B,H,I", KEEPING)
def test_a_small_unit_that_remembers_among_units_that_forget(bp, cell, T, B, H, I):
    """Usual weights, but unit 0 leaks a hundredth of its state in a step (its update gate is nearly closed) and is
    1e-6 of the others."""
    w, h0 = _inputs(cell, T, B, H, I, 1.0)
    w["x"], h0[:, 0] = 1 + 0.1 * w["x"], 0
    for k in ("w_ih", "w_hh", "b", "b_ih", "b_hh"):
        if w.get(k) is not None:
            w[k] = w[k].copy()
            w[k][::H] = 0                             # row 0, of every gate
    if cell == "rnn":
        w["w_hh"][0, 0], w["w_ih"][0] = 0.99, 1e-8
    else:
        w["b_ih"][H], w["w_ih"][2 * H] = 5.0, 1e-6
    _check_units(bp, cell, w, h0)


@pytest.mark.parametrize("cell,T,B,what", [("rnn", 30000, 8, 3.2e-9), ("rnn", 30000, 16, 1.8e-9), ("gru", 10000, 4, 1e-3)])
def test_a_unit_that_only_adds_up(bp, cell, T, B, what):
    """A unit that has hardly begun to grow in the steps before a seam: what it lacks there is less than a rounding of
    the largest state."""
    H = 20
    w, h0 = _inputs(cell, T, B, H, 1, 1.0)
    w["x"], h0[:] = np.ones_like(w["x"]), 0
    for k in ("w_ih", "w_hh", "b", "b_ih", "b_hh"):
        if w.get(k) is not None:
            w[k] = w[k].copy()
            w[k][::H] = w[k][1::H] = 0
    if cell == "rnn":
        w["w_hh"][0, 0], w["w_ih"][0], w["b"][1] = 1.0, what, 3.0
        w["b_ih"] = w["b"]
    else:
        w["b_ih"][H], w["b_ih"][2 * H], w["b_ih"][2 * H + 1] = 11.0, what, 3.0
    _check_units(bp, cell, w, h0)


@pytest.mark.parametrize("T,B", [(1000, 16), (600, 100), (400, 256)])
def test_small_units_of_a_training_iteration(bp, T, B):
    """The iteration walks in its own launch (rounds of four walks) and in those of the forward call."""
    import torch
    w, h0 = _uncoupled("rnn", T, B, 20, 1, 0.99)
    rng = np.random.default_rng(T)
    p = {"w_ih": w["w_ih"], "w_hh": w["w_hh"], "b_ih": w["b"], "b_hh": 0 * w["b"],
         "w_out": rng.uniform(-0.2, 0.2, (10, 20)).astype(np.float32), "b_out": np.zeros(10, np.float32)}
    tr = bp.RnnTrainer(T, B, 20, 1, 10, {k: to_gpu(v) for k, v in p.items()})
    tr.step(to_gpu(w["x"]), to_gpu(rng.integers(0, 10, B).astype(np.int32)))
    ref = _oracle("rnn", w, h0)
    got, base = _unit_errors(to_np(tr.h), ref), _unit_errors(_run(bp, "rnn", w, h0, PIECE), ref)
    assert np.all(got <= 2 * base + 2.0 ** -24), (got, base)
