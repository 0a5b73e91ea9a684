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


def follow_oracle(p, s, E, seed=0):
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


@pytest.mark.parametrize("wide", [0, 1])
@pytest.mark.parametrize("run,spread", [(1, 1), (2, None), (4, 0), (96, 0)])
def test_spread_copy_only_where_entries_lie_apart(run, spread, wide):
    # Columns whose entries are runs of neighbours, stored in a random order: packed, a run shares 64-byte lines.
    rng = np.random.default_rng(run)
    n, L, per = 5_000, 60_000, 96
    start = np.stack([rng.choice(L // run, per // run, replace=False) for _ in range(n)]) * run
    idx = (start[:, :, None] + np.arange(run)).reshape(n, per)
    idx = rng.permuted(idx, axis=1).astype(np.int32)
    val = (rng.standard_normal(n * per) / np.sqrt(per)).astype(np.float32)
    p = synth.Problem("runs", "ridge_primal", "csc", L, n, np.arange(n + 1, dtype=np.int64) * per, idx.reshape(-1), val,
                      rng.standard_normal(L).astype(np.float32), 1e-2, 0)
    s = scd.solver_for(p)
    s.set_option("shared_fp64", wide)
    s.set_option("window", 400)
    i = s.info()
    lines = np.mean([len(np.unique(r >> (3 if wide else 4))) for r in idx[:500]]) / per
    print(f"run {run} wide {wide}: {i['kernel']} lines per entry {lines:.3f} spread {s.get_option('next_spread')}", flush=True)
    assert i["kernel"] == "pipelined" and i["window"] == 400
    assert s.get_option("next_spread") == (lines >= (0.7 if wide else 0.47)) and spread in (None, s.get_option("next_spread"))
    follow_oracle(p, s, 2)
    s.set_option("window", 0)
    s.set_option("spread", 0)
    assert s.get_option("next_spread") == 0
    s.close()


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


# ------------------------------------------------------------- set-up statistics

def probe_signs(c, probe):
    """Rademacher sign of coordinate c in a probe (MurmurHash3 finaliser of c xor probe * golden ratio)."""
    x = (c ^ ((probe * 0x9E3779B9) & 0xFFFFFFFF)) & 0xFFFFFFFF
    x = x.astype(np.uint64)
    for shift, mul in ((16, 0x85EBCA6B), (13, 0xC2B2AE35), (16, None)):
        x ^= x >> np.uint64(shift)
        if mul is not None:
            x = (x * np.uint64(mul)) & np.uint64(0xFFFFFFFF)
    return np.where(x & np.uint64(1), 1.0, -1.0)


def reference_coupling(p):
    """(coupling, coherence) of scd_info_t in fp64 from their definition, with the library's probes."""
    seg = np.repeat(np.arange(p.C), np.diff(p.ptr))
    val = p.val.astype(np.float64)
    norms = np.bincount(seg, val * val, p.C)
    mu = 0.0 if p.form == "svm_dual" else p.lam * p.n_rows
    full = norms > 0
    scale = np.where(full, (p.y if p.form == "svm_dual" else 1.0) / np.sqrt(np.where(full, norms + mu, 1.0)), 0.0)
    diag = np.where(full, norms / np.where(full, norms + mu, 1.0), 0.0)
    a = val * scale[seg]
    ones = np.bincount(p.idx, a, p.L)
    n = full.sum()
    K = np.zeros(p.C)
    for probe in range(1, 9):
        z = probe_signs(np.arange(p.C, dtype=np.int64), probe)
        T = np.bincount(p.idx, a * z[seg], p.L)
        K += np.where(full, (np.bincount(seg, a * T[p.idx], p.C) - diag * z) ** 2, 0.0)
    return K.max() / 8 / (n - 1), (ones @ ones - diag.sum()) / (n * (n - 1))


@pytest.mark.parametrize("case", ["dense", "sparse", "dual", "text", "terms", "click", "click_hot"])
def test_coupling_estimate(case):
    # click_hot: entries beyond the 2,048 hits from which the probe sums them in LDS.
    p = {"dense": lambda: synth.make("dense_ridge"),
         "sparse": lambda: synth.make("sparse_ridge", n_rows=3_000, n_cols=2_001, density=3e-3),
         "dual": lambda: synth.as_ridge_dual(synth.make("sparse_ridge", n_rows=3_000, n_cols=2_001, density=3e-3)),
         "text": lambda: synth.make("text_svm", n_rows=700, n_cols=30_011, row_nnz=211),
         "terms": lambda: synth.make("text_ridge_csc", n_rows=5_003, n_cols=30_011, row_nnz=97),
         "click": lambda: synth.make("click_svm", n_rows=9_001, n_cols=20_011),
         "click_hot": lambda: synth.make("click_svm", n_rows=60_001, n_cols=70_001)}[case]()
    s = scd.solver_for(p)
    info = s.info()
    hits = np.bincount(p.idx, minlength=p.L)
    print(f"{case}: coupling {info['coupling']:.6e} max hits {info['max_hits']}", flush=True)
    assert info["max_hits"] == hits.max()
    assert (hits.max() >= 2048) or case != "click_hot"
    coupling, coherence = reference_coupling(p)
    # fp32 sums of up to `hits` terms, then a sum over the segment: a few 1e-6 of either
    assert abs(info["coupling"] - coupling) <= 2e-5 * coupling
    assert abs(info["coherence"] - coherence) <= 2e-5 * max(abs(coherence), coupling)
    if info["hot_entries"]:
        # the most used entries, cut where the count of hits changes
        order = np.sort(hits)[::-1]
        n = info["hot_entries"]
        assert order[n - 1] >= 1 and (n == p.L or order[n] < order[n - 1])
    s.close()


def test_coupling_estimate_without_memory_for_the_rows():
    # L so large that the probe's rows (32 bytes per shared-vector entry) do not fit what is left of
    # the GPU's memory: one probe at a time, with the same result.
    rng = np.random.default_rng(6)
    n, L, per = 2_000, 150_000_000, 20
    idx = np.sort(rng.integers(0, 300, (n, per)) * (L // 300) + np.arange(per), axis=1).astype(np.int32)
    p = synth.Problem("wide", "ridge_dual", "csr", n, L, np.arange(n + 1, dtype=np.int64) * per, idx.reshape(-1),
                      rng.standard_normal(n * per).astype(np.float32), np.ones(n, dtype=np.float32), 1e-3, 0)
    coupling, coherence = reference_coupling(p)
    got = []
    for leave in (None, 4 << 30):  # 4.8 GB of rows, 1.2 GB for everything else
        torch.cuda.empty_cache()
        free = torch.cuda.mem_get_info()[0]
        hold = torch.empty(free - leave, dtype=torch.uint8, device="cuda") if leave else None
        s = scd.solver_for(p)
        got.append((s.info()["coupling"], s.info()["coherence"]))
        s.close()
        del hold
    torch.cuda.empty_cache()
    for c, h in got:
        assert abs(c - coupling) <= 2e-5 * coupling and abs(h - coherence) <= 2e-5 * max(abs(coherence), coupling)


@pytest.mark.parametrize("case", ["fp64", "cut"])
def test_create_with_little_memory(case):
    # What scd_create holds while it runs is given up where memory is short: the counts when the shared
    # vector is allocated again in fp64 ("fp64": an index that all rows have), and the hot set that would cut
    # an automatic window of 17 to 64 ("cut"; the pipelined kernel runs it).
    if case == "fp64":
        rng = np.random.default_rng(6)
        n, L, per = 30_000, 260_000_000, 80
        idx = np.sort(rng.integers(1, 3_000, (n, per)) * (L // 3_000) + np.arange(per), axis=1).astype(np.int32)
        idx[:, 0] = 0
        p = synth.Problem("wide", "ridge_dual", "csr", n, L, np.arange(n + 1, dtype=np.int64) * per, idx.reshape(-1),
                          (rng.standard_normal(n * per) / np.sqrt(per)).astype(np.float32),
                          rng.standard_normal(n).astype(np.float32), 1e-2, 0)
        leave = 8 * L + (256 << 20)  # the vector in fp64, not the counts (4 bytes an index) beside it
    else:
        n, L = 60_000, 500_000_000
        p = synth.as_ridge_dual(synth.make("click_svm", n_rows=n, n_cols=L, lam=6 / n))
        leave = 8 * L + (400 << 20)  # the vector and the counts, not the hot set's table of 2 bytes an index
    d = scd.upload(p)
    torch.cuda.empty_cache()
    hold = torch.empty(torch.cuda.mem_get_info()[0] - leave, dtype=torch.uint8, device="cuda")
    s = scd.Solver(p.n_rows, p.n_cols, *d, p.lam, p.form)
    i = s.info()
    print(f"{case}: {i['kernel']} auto window {i['auto_window']} fp64 {i['shared_fp64']} hot {i['hot_entries']}", flush=True)
    assert i["shared_fp64"] == (case == "fp64") and i["hot_entries"] == 0 and i["kernel"] == "pipelined"
    assert case == "fp64" or 16 < i["auto_window"] <= 64
    P0, _ = s.objective()
    s.epochs(0, 2)
    assert 0.0 <= s.duality_gap() < abs(P0)
    s.close()
    del hold
    torch.cuda.empty_cache()


# ------------------------------------------------------------- hot-set plans

def test_staged_from_16_mb_of_entries():
    # 39 entries of 8 bytes a row: the first matrix above 16 MiB has 53,774 rows.
    for rows, kernel in ((53_773, "hot_lds"), (53_774, "hot_staged")):
        p = synth.make("click_svm", n_rows=rows, n_cols=70_003)
        s = scd.solver_for(p)
        info = s.info()
        print(f"{rows} rows: {info['kernel']} auto window {info['auto_window']}", flush=True)
        assert info["kernel"] == kernel
        follow_oracle(p, s, 4)
        s.close()


REPLAYED = {  # problem, options, epoch kernel
    "pipelined": (lambda: synth.make("sparse_ridge", n_rows=20_000, n_cols=10_000, density=1e-3, lam=1e-3), {"window": 300}, "pipelined"),
    "team": (lambda: synth.make("dense_ridge"), {"window": 4, "team": 4}, "team"),
    "split": (lambda: synth.make("text_ridge_csc", n_rows=3_500, n_cols=166_000, row_nnz=370), {"split_part": 128}, "split"),
    "queued": (lambda: synth.make("text_ridge_csc", n_rows=3_500, n_cols=166_000, row_nnz=370), {"split": 0}, "queued"),
    "hot": (lambda: synth.make("click_svm", n_rows=20_001, n_cols=30_001), {}, "hot_lds"),
    "staged": (lambda: synth.make("click_svm", n_rows=60_001, n_cols=70_001), {}, "hot_staged"),
}


@pytest.mark.parametrize("case", sorted(REPLAYED))
def test_epochs_replayed_from_a_graph(case):
    # A captured call of two epochs repeats their visiting orders at every replay; the oracle runs the same
    # orders.  Eager epochs and synchronisations between the replays, each checked as an eager epoch is.
    make, options, kernel = REPLAYED[case]
    p = make()
    s = scd.solver_for(p)
    for key, value in options.items():
        s.set_option(key, value)
    assert s.info()["kernel"] == kernel
    P0, _ = s.objective()
    side = torch.cuda.Stream()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side):
        s.epochs(0, 2)
    model, shared = np.zeros(p.C), np.zeros(p.L)
    for replay in range(4):
        graph.replay()
        orc.epochs(p.form, p.n_rows, p.n_cols, p.ptr, p.idx, p.val, p.y, p.lam, 0, 0, 2, model, shared)
        if replay == 1:
            torch.cuda.synchronize()
            s.set_state(*s.get_state()[:2], epoch=9)
            s.epochs(0, 1)
            orc.epochs(p.form, p.n_rows, p.n_cols, p.ptr, p.idx, p.val, p.y, p.lam, 0, 9, 1, model, shared)
        torch.cuda.synchronize()
        Gr = orc.objectives(p.form, p.n_rows, p.n_cols, p.ptr, p.idx, p.val, p.y, p.lam, model, shared)[2]
        gm, gs, _ = s.get_state()
        gm, gs = f64(gm), f64(gs)
        fresh = orc.fresh_shared(p.form, p.n_rows, p.n_cols, p.ptr, p.idx, p.val, p.y, p.lam, gm)
        assert np.max(np.abs(gs - fresh)) <= 1e-4 * np.max(np.abs(fresh)), replay
        G = s.duality_gap()
        print(f"  {case} replay {replay}: gap {G:.3e} oracle {Gr:.3e}", flush=True)
        assert G <= 2.0 * Gr + 1e-6 * abs(P0), replay
    s.close()


@pytest.mark.parametrize("wide", [0, 1])
def test_wide_automatic_window_cut_for_the_hot_set(wide):
    # The ridge dual on click rows couples weakly enough for a window between 17 and 64 at this
    # lambda; cut to 16 for the staged kernel, it follows the oracle; an explicit window, the option
    # staged = 0 and a smaller matrix keep the pipelined kernel.
    p = synth.as_ridge_dual(synth.make("click_svm", n_rows=60_000, n_cols=90_000, lam=6 / 60_000))
    s = scd.solver_for(p)
    s.set_option("shared_fp64", wide)
    auto = s.info()["auto_window"]
    print(f"auto window {auto} {s.info()['kernel']} hot {s.info()['hot_entries']}", flush=True)
    assert 16 < auto <= 64 and s.info()["kernel"] == "hot_staged" and s.info()["window"] == 16
    assert s.get_option("next_window") == 16
    follow_oracle(p, s, 4)
    assert s.get_option("next_window") == 16
    for key, value in (("window", auto), ("staged", 0), ("hot", 0), ("group", 8), ("pipeline", 0)):
        s.set_option(key, value)
        assert (s.info()["kernel"] == "hot_staged") == (key == "pipeline"), key
        s.set_option(key, {"staged": 1, "hot": 1, "pipeline": 1}.get(key, 0))
        assert s.info()["kernel"] == "hot_staged", key
    s.close()
    small = synth.as_ridge_dual(synth.make("click_svm", n_rows=40_000, n_cols=60_000, lam=6 / 40_000))
    s = scd.solver_for(small)
    assert s.info()["auto_window"] > 16 and s.info()["kernel"] == "pipelined"
    # the plan follows from the options, not from the order they are set in
    s.set_option("staged", 2)
    assert s.info()["kernel"] == "hot_staged" and s.info()["window"] == 16
    follow_oracle(small, s, 2)
    s.set_option("staged", 1)
    assert s.info()["kernel"] == "pipelined"
    s.close()


def test_hot_set_built_beside_a_running_gap_evaluation():
    # set_option("window", 8) counts hits on a stream of its own while a gap evaluation is still queued
    # behind epochs on the caller's: neither may touch the other's scratch.
    p = synth.make("sparse_ridge", n_rows=60_000, n_cols=30_000, density=5e-4, lam=1e-2)
    s, t = scd.solver_for(p), scd.solver_for(p)
    assert s.info()["hot_entries"] == 0 and s.info()["kernel"] == "pipelined"
    t.set_option("window", 8)
    want = t.info()["hot_entries"]
    assert want > 0
    stream = torch.cuda.Stream()
    torch.cuda.synchronize()
    s.epochs(0, 400, stream=stream)
    for slot in range(4):
        s.duality_gap_async(slot, stream=stream)
        s.epochs(0, 1, stream=stream)
    s.set_option("window", 8)
    got = [s.duality_gap_wait(slot) for slot in range(4)]
    torch.cuda.synchronize()
    # at the minimiser: the four evaluations differ by fp32 rounding of the state only
    P, D = s.objective()
    assert s.info()["hot_entries"] == want and s.info()["kernel"] == "hot_lds"
    for gap, Ps, Ds in got:
        assert abs(Ps - P) <= 1e-5 * abs(P) and abs(Ds - D) <= 1e-5 * abs(D) and abs(gap) <= 1e-5 * abs(P)
    s.close()
    t.close()


# ------------------------------------------------------------- passes over a frozen vector

@pytest.mark.parametrize("wide", [0, 1])
@pytest.mark.parametrize("form,rows", [("svm_dual", 215_093), ("svm_dual", 215_093 - 5), ("ridge_dual", 217_001)])
def test_frozen_passes_with_the_hot_set_in_lds(form, rows, wide):
    # 39 entries a row: the passes read the hot set from LDS from 8 Mi entries (215,093 rows) on.
    # Tolerances: a 39-term fp32 sum, 39 x 2^-24 of sum |a u|; fp64 objectives 1e-9.
    p = synth.make("click_svm", n_rows=rows, n_cols=300_007)
    p = synth.as_ridge_dual(p) if form == "ridge_dual" else p
    s = scd.solver_for(p)
    s.set_option("window", 8)  # builds the hot set whatever the automatic window is
    s.set_option("shared_fp64", wide)
    assert s.info()["hot_entries"] > 0 and (p.nnz >= 8 << 20) == (rows >= 215_093)
    rng = np.random.default_rng(8)
    u = rng.standard_normal(p.L).astype(np.float32)
    got = f64(s.gather_dots(torch.from_numpy(u).cuda()))
    ref, cond = orc.gather_dots(p.ptr, p.idx, p.val, u)
    assert np.all(np.abs(got - ref) <= 39 * 2.0 ** -24 * cond)
    model = rng.random(p.C).astype(np.float32)
    shared = (0.1 * rng.standard_normal(p.L)).astype(np.float32)
    s.set_state(torch.from_numpy(model).cuda(), torch.from_numpy(shared).cuda(), 0)
    P, D = s.objective()
    Pr, Dr, _ = orc.objectives(p.form, p.n_rows, p.n_cols, p.ptr, p.idx, p.val, p.y, p.lam, model.astype(np.float64),
                               shared.astype(np.float64))
    scale = max(abs(Pr), abs(Dr))
    assert abs(P - Pr) <= 1e-9 * scale and abs(D - Dr) <= 1e-9 * scale
    s.close()


@pytest.mark.parametrize("kind", ["hot", 3, 17, 49, 161, 300])
def test_gather_dots_of_infinities(kind):
    # u with infinities and NaN: a segment sees those of its own entries and no others, also where lanes
    # past its end stand in with its first entry.  Each reference sum is the one of IEEE arithmetic.
    rng = np.random.default_rng(12)
    if kind == "hot":
        p = synth.make("click_svm", n_rows=215_093, n_cols=300_007)
        s = scd.solver_for(p)
        s.set_option("window", 8)
        assert s.info()["hot_entries"] > 0
    else:
        n, L = 1_003, 4_099
        lens = np.concatenate([[0, 1, 2], rng.integers(max(1, kind - 2), kind + 3, n - 3)])
        ptr = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
        idx = np.concatenate([np.sort(rng.choice(L, k, replace=False)) for k in lens]).astype(np.int32)
        val = rng.standard_normal(int(ptr[-1])).astype(np.float32)
        p = synth.Problem("lengths", "ridge_dual", "csr", n, L, ptr, idx, val, np.ones(n, dtype=np.float32), 1e-2, 0)
        s = scd.solver_for(p)
    u = rng.standard_normal(p.L).astype(np.float32)
    first = p.idx[p.ptr[:-1][np.diff(p.ptr) > 0]]  # what the stand-in lanes would read
    u[rng.choice(first, 8)] = np.inf
    u[rng.choice(first, 8)] = -np.inf
    u[rng.integers(0, p.L, 2)] = np.nan
    got = f64(s.gather_dots(torch.from_numpy(u).cuda()))
    seg = np.repeat(np.arange(p.C), np.diff(p.ptr))
    with np.errstate(invalid="ignore"):
        ref = np.bincount(seg, p.val.astype(np.float64) * u[p.idx], p.C)
    bad = ~np.isfinite(ref)
    print(f"{kind}: {np.isinf(ref).sum()} infinite, {np.isnan(ref).sum()} NaN of {p.C}", flush=True)
    assert np.isinf(ref).any() and np.array_equal(got[bad], ref[bad], equal_nan=True)
    cond = np.bincount(seg, np.abs(p.val.astype(np.float64) * np.where(np.isfinite(u), u, 0.0)[p.idx]), p.C)
    assert np.all(np.abs(got[~bad] - ref[~bad]) <= 600 * 2.0 ** -24 * cond[~bad])
    s.close()


@pytest.mark.parametrize("per", [3, 17, 49, 161, 300])
def test_gather_dots_over_segment_lengths(per):
    # the group widths 4 to 64, segments from empty to beyond one block of each
    rng = np.random.default_rng(per)
    n, L = 1_003, 4_099
    lens = np.concatenate([[0, 1, 2, 3, 600, 0], rng.integers(max(1, per - 2), per + 3, n - 6)])
    ptr = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    idx = np.concatenate([np.sort(rng.choice(L, k, replace=False)) for k in lens]).astype(np.int32)
    val = rng.standard_normal(int(ptr[-1])).astype(np.float32)
    p = synth.Problem("lengths", "ridge_dual", "csr", n, L, ptr, idx, val, rng.standard_normal(n).astype(np.float32), 1e-2, 0)
    s = scd.solver_for(p)
    u = rng.standard_normal(L).astype(np.float32)
    got = f64(s.gather_dots(torch.from_numpy(u).cuda()))
    ref, cond = orc.gather_dots(ptr, idx, val, u)
    assert np.all(np.abs(got - ref) <= 600 * 2.0 ** -24 * cond) and got[0] == 0.0
    model = rng.standard_normal(n).astype(np.float32)
    s.set_state(torch.from_numpy(model).cuda(), torch.from_numpy(u).cuda(), 0)
    P, D = s.objective()
    Pr, Dr, _ = orc.objectives(p.form, n, L, ptr, idx, val, p.y, p.lam, model.astype(np.float64), u.astype(np.float64))
    scale = max(abs(Pr), abs(Dr))
    assert abs(P - Pr) <= 1e-9 * scale and abs(D - Dr) <= 1e-9 * scale
    s.close()


# ------------------------------------------------------------- lockstep kernel

def _rows(lens, L, form, lam, seed, repeat=False, positive=False):
    """Random segments of the given lengths over L shared indices (the upper fifth unused)."""
    rng = np.random.default_rng(seed)
    used = L - L // 5
    n = len(lens)
    ptr = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    idx = np.concatenate([np.sort(rng.choice(used, k, replace=repeat)) for k in lens]).astype(np.int32)
    val = rng.standard_normal(int(ptr[-1])) / np.sqrt(np.repeat(np.maximum(lens, 1), lens))
    val = (np.abs(val) if positive else val).astype(np.float32)
    rows, cols = (L, n) if form == "ridge_primal" else (n, L)
    y = rng.standard_normal(rows).astype(np.float32)
    y = np.where(y < 0, -1.0, 1.0).astype(np.float32) if form == "svm_dual" else y
    return synth.Problem("rows", form, "csc" if form == "ridge_primal" else "csr", rows, cols, ptr, idx, val, y, lam, 0)


def _lockstep(s):
    """The lockstep kernel runs the epochs, with the whole automatic window."""
    i = s.info()
    lock = s.get_option("next_lockstep") == 1
    assert not lock or (i["kernel"] == "pipelined" and i["group_lanes"] == 256 and i["window"] == i["auto_window"] <= 16)
    return lock


LOCKSTEP = {
    # (lengths, L, form): a member's part is about an eighth of a segment; 256 entries stay in registers
    "dense": lambda: synth.make("dense_ridge", n_rows=1_999, n_cols=203),
    "dense_long": lambda: synth.make("dense_ridge", n_rows=3_001, n_cols=101),  # parts of 376
    "text": lambda: synth.make("text_svm", n_rows=3_500, n_cols=166_000, row_nnz=370),
    "svm_ragged": lambda: _rows(np.concatenate([[0, 1, 2, 63, 64, 65, 0], np.full(200, 511), [2_048, 2_056, 3_000]]), 6_007,
                                "svm_dual", 1 / 210, 1),
    "dual": lambda: _rows(np.full(251, 400), 4_501, "ridge_dual", 1e-3, 2),
    "doubled": lambda: _rows(np.full(243, 330), 2_500, "ridge_primal", 1e-3, 3, repeat=True),  # repeated indices
}


@pytest.mark.parametrize("wide", [0, 1])
@pytest.mark.parametrize("case", sorted(LOCKSTEP))
def test_lockstep_follows_the_oracle(case, wide):
    p = LOCKSTEP[case]()
    s = scd.solver_for(p)
    s.set_option("shared_fp64", wide)
    info = s.info()
    print(f"{case} wide {wide}: auto window {info['auto_window']} kernel {info['kernel']} window {info['window']}", flush=True)
    assert _lockstep(s) and info["window"] >= 2
    follow_oracle(p, s, 6)
    model = f64(s.get_state()[0])
    empty = np.diff(p.ptr) == 0
    assert np.all(model[empty] == (1.0 if p.form == "svm_dual" else 0.0))
    s.set_option("lockstep", 0)
    assert not _lockstep(s)
    s.close()


@pytest.mark.parametrize("form,n,lam", [("ridge_primal", 243, 1e-3), ("ridge_dual", 243, 1e-3), ("svm_dual", 120, 1 / 120)])
def test_lockstep_not_of_coherent_coordinates(form, n, lam):
    # Positive values (and one label): the coordinates of a round would overshoot together.  The same values
    # with random signs run in lockstep.
    for positive in (True, False):
        p = _rows(np.full(n, 330), 2_500, form, lam, 3, positive=positive)
        if form == "svm_dual":
            p.y[:] = 1.0
        s = scd.solver_for(p)
        i = s.info()
        pull = (i["auto_window"] - 1) * i["coherence"]
        print(f"{form} positive {positive}: auto window {i['auto_window']} coherence {i['coherence']:.4f} ({pull:.3f})", flush=True)
        assert 2 <= i["auto_window"] <= 16 and (pull > 0.1) == positive and _lockstep(s) == (not positive)
        if not positive:
            follow_oracle(p, s, 4)
        s.close()


def test_lockstep_converges_and_resumes():
    # to the normal equations (condition about 4: 40 epochs reach fp32 rounding), over several calls
    # and a state written back in between
    p = synth.make("dense_ridge", n_rows=2_000, n_cols=200)
    A = np.zeros((p.n_rows, p.n_cols))
    for m in range(p.n_cols):
        A[p.idx[p.ptr[m]:p.ptr[m + 1]], m] = p.val[p.ptr[m]:p.ptr[m + 1]]
    star = np.linalg.solve(A.T @ A + p.n_rows * p.lam * np.eye(p.n_cols), A.T @ p.y.astype(np.float64))
    s = scd.solver_for(p)
    assert _lockstep(s)
    s.epochs(0, 17)
    s.set_state(*s.get_state())
    s.epochs(0, 1)
    s.epochs(0, 22)
    got = f64(s.get_state()[0])
    assert s.info()["epoch"] == 40 and np.max(np.abs(got - star)) <= 1e-4 * np.max(np.abs(star))
    s.close()


@pytest.mark.parametrize("wide", [0, 1])
def test_lockstep_of_an_infinite_entry(wide):
    # A state with one infinite shared-vector entry: the coordinate that has it diverges, the others reach
    # the minimiser as without it (condition about 5: 40 epochs reach fp32 rounding).  It is the first cell of
    # a member, and every part leaves lanes without an entry.
    rng = np.random.default_rng(14)
    n, per, L = 251, 400, 4_501
    idx = np.stack([np.sort(rng.choice(np.arange(500, L), per, replace=False)) for _ in range(n)]).astype(np.int32)
    idx[0] = np.arange(per)  # apart from all others
    p = synth.Problem("apart", "ridge_dual", "csr", n, L, np.arange(n + 1, dtype=np.int64) * per, idx.reshape(-1),
                      (rng.standard_normal(n * per) / 20).astype(np.float32), rng.standard_normal(n).astype(np.float32), 1e-3, 0)
    out = []
    for first in (0.0, np.inf):
        s = scd.solver_for(p)
        s.set_option("shared_fp64", wide)
        assert _lockstep(s)
        shared = torch.zeros(L, device="cuda")
        shared[0] = first
        s.set_state(torch.zeros(n, device="cuda"), shared, 0)
        s.epochs(0, 40)
        m, u, _ = s.get_state()
        out.append((f64(m), f64(u)))
        s.close()
    (m0, u0), (m1, u1) = out
    assert np.all(np.isfinite(m0)) and not np.isfinite(m1[0]) and not np.any(np.isfinite(u1[:per]))
    assert np.max(np.abs(m1[1:] - m0[1:])) <= 1e-4 * np.max(np.abs(m0))
    assert np.max(np.abs(u1[per:] - u0[per:])) <= 1e-4 * np.max(np.abs(u0))


def test_lockstep_selection():
    p = LOCKSTEP["text"]()
    s = scd.solver_for(p)
    assert _lockstep(s) and s.get_option("lockstep") == 1
    for key, value in (("lockstep", 0), ("group", 256), ("pipeline", 0), ("fresh_reads", 1), ("team", 0), ("window", 1)):
        before = s.get_option(key)
        s.set_option(key, value)
        assert not _lockstep(s), key
        s.epochs(0, 1)
        s.set_option(key, before)
        assert _lockstep(s), key
    for bad in (-1, 2):
        with pytest.raises(scd.ScdError):
            s.set_option("lockstep", bad)
    gm, gs, _ = s.get_state()
    fresh = orc.fresh_shared(p.form, p.n_rows, p.n_cols, p.ptr, p.idx, p.val, p.y, p.lam, f64(gm))
    assert np.max(np.abs(f64(gs) - fresh)) <= 1e-4 * np.max(np.abs(fresh))
    s.close()
    # used entries that eight workgroups' LDS holds (8 x 20,471), and more: 256 rows of 200 common indices and
    # their own
    rng = np.random.default_rng(5)
    n = 256
    for own, fits in ((638, True), (640, False)):
        used = 200 + n * own
        idx = np.concatenate([np.broadcast_to(np.arange(200), (n, 200)),
                              200 + np.arange(n)[:, None] + n * np.arange(own)[None, :]], axis=1).astype(np.int32)
        per = 200 + own
        q = synth.Problem("wide", "ridge_dual", "csr", n, used, np.arange(n + 1, dtype=np.int64) * per, idx.reshape(-1),
                          (rng.standard_normal(n * per) / np.sqrt(per)).astype(np.float32),
                          rng.standard_normal(n).astype(np.float32), 1 / n, 0)
        s = scd.solver_for(q)
        i = s.info()
        print(f"{used} used entries: kernel {i['kernel']} window {i['window']} auto {i['auto_window']}", flush=True)
        assert 2 <= i["auto_window"] <= 16 and _lockstep(s) == fits == (used <= 8 * 20_471)
        follow_oracle(q, s, 2)
        s.close()


@pytest.mark.parametrize("n,L,common,seed", [(64, 1_025, 60, 1), (96, 60_007, 200, 2), (270, 111_000, 300, 3), (250, 300_001, 0, 4)])
def test_lockstep_ranges_and_cells(n, L, common, seed):
    # The members' index ranges come from the hits: cut where the entries are about equal, or, where
    # that exceeds a member's LDS (seed 3: 23,625 entries a member, most of an index of their own), where the cells are.  A cell given twice or to the wrong member breaks the invariant at its indices.
    rng = np.random.default_rng(seed)
    per = 700 if seed == 3 else 450
    own = (L - common) // n if seed == 3 else 0
    idx = []
    for r in range(n):
        a = np.arange(common)
        m = per - common
        if own:  # every other index belongs to one row only
            b = common + r + n * rng.choice(own, m, replace=False)
        else:
            b = common + rng.choice(L - common - 3, m, replace=False)  # the last indices unused
        idx.append(np.sort(np.concatenate([a, b])))
    lens = np.array([len(i) for i in idx])
    ptr = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    val = (rng.standard_normal(int(ptr[-1])) / np.sqrt(per)).astype(np.float32)
    p = synth.Problem("ranges", "ridge_dual", "csr", n, L, ptr, np.concatenate(idx).astype(np.int32), val,
                      rng.standard_normal(n).astype(np.float32), 1 / n, 0)
    s = scd.solver_for(p)
    i = s.info()
    print(f"{n} x {L}: auto window {i['auto_window']} window {i['window']} used {len(np.unique(p.idx))}", flush=True)
    assert _lockstep(s)
    follow_oracle(p, s, 4)
    # every index some entry points at takes part, and no other changes
    gs = f64(s.get_state()[1])
    assert np.all(gs[np.setdiff1d(np.arange(L), p.idx)] == 0.0) and np.mean(gs[np.unique(p.idx)] != 0.0) > 0.999
    s.close()


@pytest.mark.parametrize("case,lockstep", [("even", True), ("half_range", True), ("one_range", False), ("few_long", True),
                                           ("many_long", True), ("long", False)])
def test_lockstep_of_uneven_parts(case, lockstep):
    # Parts of up to 256 and of up to 512 entries stay in registers.  Beyond, the longest part of a round holds
    # up the others: rows that lie in one of the eight index ranges, and long rows among short ones, keep the
    # pipelined kernel; a few do not matter.  (250 weakly coupled rows: a window of 250 / 16.)
    rng = np.random.default_rng(21)
    n, L = 250, 60_000
    tenth = rng.random(n) < 0.1
    per, span = {"even": (700, L), "half_range": (500, 520), "one_range": (700, 800), "few_long": (330, L),
                 "many_long": (np.where(tenth, 3_000, 330), L), "long": (np.where(tenth, 6_000, 330), L)}[case]
    lens = np.broadcast_to(per, n).copy()
    if case == "few_long":
        lens[100] = 1_500
    idx = np.concatenate([np.sort(rng.integers(0, L - span + 1) + rng.choice(span, m, replace=False)) for m in lens])
    val = (rng.standard_normal(len(idx)) / np.sqrt(np.repeat(lens, lens))).astype(np.float32)
    p = synth.Problem("uneven", "ridge_dual", "csr", n, L, np.concatenate([[0], np.cumsum(lens)]).astype(np.int64),
                      idx.astype(np.int32), val, rng.standard_normal(n).astype(np.float32), 1 / n, 0)
    s = scd.solver_for(p)
    i = s.info()
    print(f"{case}: auto window {i['auto_window']} window {i['window']} entries {p.nnz}", flush=True)
    assert i["auto_window"] == 15 and i["kernel"] == "pipelined" and _lockstep(s) == lockstep
    follow_oracle(p, s, 4)
    s.close()


def test_lockstep_limits_on_the_entries_in_flight():
    # 24,576 entries in flight while the copy takes at most 2.5 MB (6 bytes an entry), else 12,288
    for rows, cols in ((2_000, 208), (2_000, 209), (2_500, 375), (6_000, 100)):
        p = synth.make("dense_ridge", n_rows=rows, n_cols=cols)
        s = scd.solver_for(p)
        i = s.info()
        in_flight = i["auto_window"] * rows
        want = 2 <= i["auto_window"] <= 16 and in_flight <= (24_576 if p.nnz * 6 <= 2_500_000 else 12_288)
        print(f"{rows} x {cols}: auto {i['auto_window']} in flight {in_flight} window {i['window']}", flush=True)
        assert i["kernel"] == "pipelined" and _lockstep(s) == want
        assert i["window"] == (i["auto_window"] if want else i["auto_window"] * 4 // 5)
        follow_oracle(p, s, 3)
        s.close()


def test_lockstep_handles_side_by_side():
    # two solvers on two streams, epochs enqueued together: each follows its own problem
    p, q = LOCKSTEP["text"](), LOCKSTEP["dual"]()
    streams = [torch.cuda.Stream() for _ in range(2)]
    solvers = [scd.solver_for(x) for x in (p, q)]
    torch.cuda.synchronize()
    for _ in range(5):
        for s, st in zip(solvers, streams):
            s.epochs(0, 3, stream=st)
    torch.cuda.synchronize()
    for x, s in zip((p, q), solvers):
        gm, gs, e = s.get_state()
        assert e == 15 and s.duality_gap() >= 0.0
        fresh = orc.fresh_shared(x.form, x.n_rows, x.n_cols, x.ptr, x.idx, x.val, x.y, x.lam, f64(gm))
        assert np.max(np.abs(f64(gs) - fresh)) <= 1e-4 * np.max(np.abs(fresh))
        s.close()


def test_kernels_with_waits_between_workgroups_side_by_side():
    # Epochs of lockstep, team (256 workgroups) and staged solvers queued on streams of their own: whatever
    # workgroups are resident first, every epoch ends and no wait times out.
    team = synth.make("dense_ridge", n_rows=4_000, n_cols=300)
    problems = [LOCKSTEP["text"](), team, synth.make("click_svm", n_rows=60_001, n_cols=70_001), LOCKSTEP["dual"]()]
    solvers = [scd.solver_for(p) for p in problems]
    solvers[1].set_option("window", 16)
    solvers[1].set_option("team", 16)
    assert [s.info()["kernel"] for s in solvers] == ["pipelined", "team", "hot_staged", "pipelined"]
    assert _lockstep(solvers[0]) and _lockstep(solvers[3])
    streams = [torch.cuda.Stream() for _ in solvers]
    torch.cuda.synchronize()
    for _ in range(6):
        for s, st in zip(solvers, streams):
            s.epochs(0, 5, stream=st)
    torch.cuda.synchronize()
    for p, s in zip(problems, solvers):
        gm, gs, e = s.get_state()
        assert e == 30 and s.duality_gap() >= 0.0  # raises where a wait timed out
        fresh = orc.fresh_shared(p.form, p.n_rows, p.n_cols, p.ptr, p.idx, p.val, p.y, p.lam, f64(gm))
        assert np.max(np.abs(f64(gs) - fresh)) <= 1e-4 * np.max(np.abs(fresh)), p.form
        s.close()


def test_lockstep_replayed_from_a_graph():
    # A captured call of two epochs repeats their visiting orders at every replay.  Replays between eager
    # epochs and state reads follow a solver that runs the same orders eagerly: the steps are the same, and
    # only the order of fp64 adds within a round differs.
    p = LOCKSTEP["text"]()
    s, t = scd.solver_for(p), scd.solver_for(p)
    assert _lockstep(s)
    zeros = torch.zeros(p.C, device="cuda"), torch.zeros(p.L, device="cuda")
    side = torch.cuda.Stream()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    s.set_state(*zeros, 0)
    torch.cuda.synchronize()
    with torch.cuda.graph(graph, stream=side):
        s.epochs(0, 2)
    for replay in range(4):
        graph.replay()
        t.set_state(*(zeros if replay == 0 else t.get_state()[:2]), epoch=0)
        t.epochs(0, 2)
        if replay == 1:  # an eager epoch between the replays
            for x in (s, t):
                x.set_state(epoch=7)
                x.epochs(0, 1)
        torch.cuda.synchronize()
        a, b = s.get_state(), t.get_state()
        assert s.duality_gap() > 0.0
        for x, y in zip(a[:2], b[:2]):
            assert float((x - y).abs().max()) <= 1e-4 * float(y.abs().max()), replay
    for x in (s, t):
        x.close()


def test_lockstep_wait_limit():
    # bounded waits with a limit of one poll: either every exchange completes in time (valid state) or
    # the timeout is reported at the next synchronising call and a written state replaces the invalid one
    p = LOCKSTEP["text"]()
    s = scd.solver_for(p)
    assert _lockstep(s)
    s.set_option("hot_wait_limit", 1)
    s.epochs(0, 3)
    try:
        s.duality_gap()
        timed_out = False
    except scd.ScdError as e:
        assert "timed out" in str(e)
        timed_out = True
    print(f"lockstep wait limit 1: timed out {timed_out}", flush=True)
    s.set_option("hot_wait_limit", 0)
    s.set_state(torch.zeros(p.C, device="cuda"), torch.zeros(p.L, device="cuda"), 0)
    follow_oracle(p, s, 3)
    s.close()
