"""Launch plans against the oracle, at the sizes where a plan's rule changes its mind.

Tolerances as in test_gpu_parity.py: |w - A model|_inf / |w|_inf <= 1e-4 after every epoch with
A model fresh in fp64, gap within 2x of the sequential oracle's plus the fp32 floor 1e-6 P(0).
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

from oracle import oracle as orc  # noqa: E402
from paper_1702_07005_amd import scd, synth  # noqa: E402


def f64(t):
    return t.detach().cpu().numpy().astype(np.float64)


def follow_oracle(p, s, E, seed=0, gate=True):
    """E epochs of `s` from the zero state, each checked against the sequential oracle."""
    model, shared = np.zeros(p.C), np.zeros(p.L)
    P0, _ = s.objective()
    for e in range(E):
        orc.epochs(p.form, p.n_rows, p.n_cols, p.ptr, p.idx, p.val, p.y, p.lam, seed, e, 1, model, shared)
        Gr = orc.objectives(p.form, p.n_rows, p.n_cols, p.ptr, p.idx, p.val, p.y, p.lam, model, shared)[2]
        s.epochs(seed, 1)
        gm, gs, _ = s.get_state()
        gm, gs = f64(gm), f64(gs)
        fresh = orc.fresh_shared(p.form, p.n_rows, p.n_cols, p.ptr, p.idx, p.val, p.y, p.lam, gm)
        assert np.max(np.abs(gs - fresh)) <= 1e-4 * max(np.max(np.abs(fresh)), 1e-30), e
        if p.form == "svm_dual":
            assert gm.min() >= 0.0 and gm.max() <= 1.0
        G = s.duality_gap()
        print(f"  epoch {e + 1}: gap {G:.3e} oracle {Gr:.3e}", flush=True)
        if gate:
            assert G <= 2.0 * Gr + 1e-6 * abs(P0), (e, G, Gr)


# ------------------------------------------------------------- lanes per coordinate, spread copy

# 256 CUs x 3 waves x 64 lanes = 49,152 lanes: a wave per coordinate up to 768 in flight, 32 lanes up
# to 1,536, 16 up to 3,072, then the fewest that hold a segment (4 lanes for these rows of 10, 8 for
# the columns of 20).
@pytest.mark.parametrize("wide", [0, 1])
@pytest.mark.parametrize("form,window,lanes", [
    ("ridge_dual", 40, 64), ("ridge_dual", 768, 64), ("ridge_dual", 769, 32), ("ridge_dual", 1536, 32),
    ("ridge_dual", 1537, 16), ("ridge_dual", 3073, 8), ("ridge_dual", 6145, 4),
    ("ridge_primal", 768, 64), ("ridge_primal", 3072, 16), ("ridge_primal", 6145, 8)])
def test_wide_groups_and_spread_copy(form, window, lanes, wide):
    p = synth.make("sparse_ridge", n_rows=20_000, n_cols=10_000, density=1e-3, lam=1e-2)
    p = synth.as_ridge_dual(p) if form == "ridge_dual" else p
    out = {}
    for spread in (1, 0):
        s = scd.solver_for(p)
        s.set_option("shared_fp64", wide)
        s.set_option("spread", spread)
        s.set_option("window", window)
        info = s.info()
        print(f"{form} window {window} wide {wide} spread {spread}: {info['kernel']} {info['group_lanes']}", flush=True)
        assert info["kernel"] == "pipelined" and info["group_lanes"] == lanes and info["window"] == window
        follow_oracle(p, s, 3)
        out[spread] = f64(s.get_state()[1])
        s.close()
    # Strongly regularised (lambda N = 200 against unit rows): after three epochs both runs are at
    # the minimiser to fp32 rounding, about sqrt(hits x epochs) 2^-24 of an entry.
    assert np.max(np.abs(out[0] - out[1])) <= 1e-5 * np.max(np.abs(out[0]))


def test_wide_groups_with_segments_of_every_length():
    # segments from empty to beyond a wave's register slices (64 x 4 entries)
    rng = np.random.default_rng(4)
    base = synth.make("sparse_ridge", n_rows=20_000, n_cols=2_000, density=1e-3)
    lens = np.concatenate([[0, 1, 63, 64, 65, 255, 256, 257, 300, 0], rng.integers(80, 161, 1_990)])
    ptr = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    idx = np.concatenate([np.sort(rng.choice(20_000, n, replace=False)) for n in lens]).astype(np.int32)
    val = rng.standard_normal(int(ptr[-1])).astype(np.float32) / 10
    p = synth.Problem("lengths", "ridge_primal", "csc", 20_000, 2_000, ptr, idx, val, base.y, 1e-3, 0)
    s = scd.solver_for(p)
    s.set_option("window", 100)
    info = s.info()
    assert info["kernel"] == "pipelined" and info["group_lanes"] == 64
    follow_oracle(p, s, 4)
    gm = f64(s.get_state()[0])
    assert gm[0] == 0.0 and gm[9] == 0.0 and np.all(gm[1:9] != 0.0)
    s.close()
