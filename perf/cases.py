"""What a user of this library has it do, as cases whose time can be taken on one GPU.

Every case is one call path of the public entry points (``paper_1702_07005_amd.scd``) on a seeded
synthetic matrix of the kind that path is used on.  ``listed`` holds the cases themselves, ``draw``
gives further ones of the same ranges, ``prepare`` makes on the GPU what a program holds before the
call, ``run`` is the call, ``work`` counts what it cannot do without, ``tolerance`` says how closely
two correct runs agree, and ``exact`` computes the same outputs in 64 bits with plain torch.

The call paths:

``train``      epochs from the zero state, then both objectives and the state: a whole fit.
``resume``     the same from a checkpoint (a state that some epochs have reached): what a training
               loop does for most of its life.
``objective``  both objectives of a state: the convergence check of a training loop.
``score``      inner products of all segments with a vector (predictions for new examples).
``create``     making a solver: validation, norms, coupling estimate, tables; then its norms.

The matrices:

``dense``      all entries N(0,1).
``uniform``    entries spread evenly with a given density, values N(0,1), unit rows.
``text``       term counts: column popularity follows Zipf(1.1), values exp(N(0,1)), unit rows.
``click``      39 one-hot fields, field sizes proportional to f^-1.2, values inside a field
               Zipf(1.2), unit rows, 3 % positive labels.
"""
import math

import torch

from paper_1702_07005_amd import scd

FIELDS = 39
EPOCH_SEED = 7  # of the visiting order


# --------------------------------------------------------------------------- inputs


def _generator(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return g


def _pointers(counts):
    ptr = torch.zeros(counts.numel() + 1, dtype=torch.int64, device="cuda")
    torch.cumsum(counts, 0, out=ptr[1:])
    return ptr


def _chunks(ptr, most=1 << 27):
    """Ranges of segments of about ``most`` entries each."""
    total, n = int(ptr[-1]), ptr.numel() - 1
    parts = max(1, -(-total // most))
    cuts = torch.searchsorted(ptr, torch.arange(1, parts, device="cuda") * (total // parts)).tolist()
    edges = sorted({0, n, *(min(n, c) for c in cuts)})
    return list(zip(edges[:-1], edges[1:]))


def _segment_of(ptr, a, b):
    """The segment of every entry of segments a..b-1, and that entry's place in it."""
    counts = ptr[a + 1:b + 1] - ptr[a:b]
    base, n = int(ptr[a]), int(ptr[b] - ptr[a])
    seg = torch.repeat_interleave(torch.arange(a, b, device="cuda"), counts, output_size=n)
    return seg, torch.arange(base, base + n, device="cuda") - ptr[seg]


def _even_indices(ptr, length, g, idx):
    """Segment k gets its entries' indices spread over [0, length): one in each of its equal parts,
    increasing and distinct."""
    for a, b in _chunks(ptr):
        seg, j = _segment_of(ptr, a, b)
        k = (ptr[seg + 1] - ptr[seg]).double()
        u = torch.rand(seg.numel(), dtype=torch.float64, device="cuda", generator=g)
        at = ((j + u) * ((length - k + 1) / k)).floor().long() + j
        idx[int(ptr[a]):int(ptr[b])] = at.clamp_(max=length - 1).int()


def _term_shares(cols, per, s=1.1):
    """The share of rows that hold each rank, so that a row holds ``per`` of the ``cols`` ranks: that
    of drawing ranks from Zipf(s) until so many distinct ones are there."""
    weight = torch.arange(1, cols + 1, dtype=torch.float64, device="cuda").pow_(-s)
    lo, hi = 1e-3, 1e9
    for _ in range(60):
        c = math.sqrt(lo * hi)
        lo, hi = (c, hi) if -float(torch.expm1(-c * weight).sum()) < per else (lo, c)
    return torch.expm1_(weight.mul_(-c)).neg_()


def _scatter(rank, n):
    """Rank to column: an affine bijection, so that popular columns lie apart."""
    step = int(0.6180339887 * n) | 1
    while math.gcd(step, n) != 1:
        step += 2
    return (rank * step + 12345) % n


def _text_rows(rows, cols, per, g, idx, val):
    share = _term_shares(cols, per)
    # in whole numbers, so that the sums are the same every time
    upto = (torch.cumsum((share * 2.0 ** 40).long(), 0).double() * 2.0 ** -40).clamp_(max=per)
    step = max(1, (1 << 26) // per)
    j = torch.arange(per, device="cuda")
    for r in range(0, rows, step):
        n = min(step, rows - r)
        # one rank from each of ``per`` ranges of equal expected count; as no share is above 1, the
        # place along the ranks grows by at least one from range to range: the ranks are distinct
        t = j + torch.rand(n, per, dtype=torch.float64, device="cuda", generator=g)
        k = torch.searchsorted(upto, t).clamp_(max=cols - 1)
        at = k + (1 - (upto[k] - t) / share[k]).clamp_(0, 1)
        rank = ((at - t).clamp_(min=0).floor().long() + j).clamp_(max=cols - 1)
        idx[r * per:(r + n) * per] = _scatter(rank, cols).int().sort(dim=1).values.view(-1)
        v = torch.randn(n, per, device="cuda", generator=g).exp_()
        val[r * per:(r + n) * per] = (v / v.double().square().sum(1, keepdim=True).sqrt()).float().view(-1)


def _click_rows(rows, cols, g, idx, val):
    share = [(f + 1) ** -1.2 for f in range(FIELDS)]
    sizes = [max(2, int(cols * s / sum(share))) for s in share]
    sizes[0] += cols - sum(sizes)
    grid, at = idx.view(rows, FIELDS), 0
    for f, n in enumerate(sizes):
        u = torch.rand(rows, dtype=torch.float64, device="cuda", generator=g)
        first, last = 0.5 ** -0.2, (n + 0.5) ** -0.2
        rank = (first - u * (first - last)).pow_(-5).sub_(0.5).floor_().long().clamp_(0, n - 1)
        grid[:, f] = (at + _scatter(rank, n)).int()
        at += n
    val.fill_(FIELDS ** -0.5)


def _by_index(ptr, idx, v, length):
    """Sums of v over the entries of each index, the same for any order of the adds (fixed point)."""
    acc = torch.zeros(length, dtype=torch.int64, device="cuda")
    for a, b in _chunks(ptr):
        s = slice(int(ptr[a]), int(ptr[b]))
        acc.index_add_(0, idx[s], (v(s, a, b).double() * 2.0 ** 32).round().long())
    return acc.double() * 2.0 ** -32


def _matrix(case, seed):
    """(rows, cols, ptr, idx, val, y) of a case, made on the GPU from the seed alone."""
    g = _generator(seed)
    rows, cols, per, kind = case["rows"], case["cols"], case["per"], case["matrix"]
    by_cols = case["form"] == "ridge_primal"
    n_seg, length = (cols, rows) if by_cols else (rows, cols)
    if kind == "dense":
        counts = torch.full((n_seg,), length, dtype=torch.int64, device="cuda")
    elif kind == "uniform":
        p = per / cols
        counts = torch.randn(n_seg, dtype=torch.float64, device="cuda", generator=g)
        counts = (length * p + counts * math.sqrt(length * p * (1 - p))).round().clamp_(0, length).long()
    elif kind == "text" and by_cols:
        share = torch.empty(cols, dtype=torch.float64, device="cuda")
        share[_scatter(torch.arange(cols, device="cuda"), cols)] = _term_shares(cols, per)
        counts = share * rows + torch.rand(cols, dtype=torch.float64, device="cuda", generator=g)
        counts = counts.floor().clamp_(max=rows).long()
    else:
        counts = torch.full((n_seg,), per, dtype=torch.int64, device="cuda")
    ptr = _pointers(counts)
    nnz = int(ptr[-1])
    idx = torch.empty(nnz, dtype=torch.int32, device="cuda")
    val = torch.empty(nnz, dtype=torch.float32, device="cuda")
    if kind == "text" and not by_cols:
        _text_rows(rows, cols, per, g, idx, val)
    elif kind == "click":
        _click_rows(rows, cols, g, idx, val)
    else:
        _even_indices(ptr, length, g, idx)
        for s in range(0, nnz, 1 << 27):
            v = val[s:s + (1 << 27)]
            v.normal_(generator=g)
            if kind == "text":
                v.exp_()
    if kind in ("uniform", "text") and (by_cols or kind == "uniform"):  # unit rows
        for a, b in _chunks(ptr):
            s = slice(int(ptr[a]), int(ptr[b]))
            if by_cols:
                if a == 0:
                    norm = _by_index(ptr, idx, lambda s, a, b: val[s].square(), rows).clamp_(min=1e-12).rsqrt_()
                val[s] = (val[s] * norm[idx[s]]).float()
            else:
                seg = _segment_of(ptr, a, b)[0]
                n2 = torch.zeros(b - a, dtype=torch.int64, device="cuda")
                n2.index_add_(0, seg - a, (val[s].double().square() * 2.0 ** 32).round().long())
                val[s] = (val[s] * (n2.double() * 2.0 ** -32).clamp_(min=1e-12).rsqrt_()[seg - a]).float()
    if kind == "click":
        y = (torch.rand(rows, device="cuda", generator=g) < 0.03).float() * 2 - 1
    else:
        plane = torch.randn(cols, device="cuda", generator=g)
        if kind == "text":
            plane *= torch.rand(cols, device="cuda", generator=g) < 0.01
        if by_cols:
            y = _by_index(ptr, idx, lambda s, a, b: val[s] * plane[_segment_of(ptr, a, b)[0]], rows)
        else:
            y = torch.zeros(rows, dtype=torch.int64, device="cuda")
            for a, b in _chunks(ptr):
                s = slice(int(ptr[a]), int(ptr[b]))
                q = (val[s].double() * plane[idx[s]] * 2.0 ** 32).round().long()
                y.index_add_(0, _segment_of(ptr, a, b)[0], q)
            y = y.double() * 2.0 ** -32
        if kind == "text":
            flip = torch.rand(rows, device="cuda", generator=g) < 0.05
            y = (torch.where(y < 0, -1.0, 1.0) * torch.where(flip, -1.0, 1.0)).float()
        else:
            y = (y + 0.01 * torch.randn(rows, dtype=torch.float64, device="cuda", generator=g)).float()
    return rows, cols, ptr, idx, val, y


# --------------------------------------------------------------------------- cases


def _case(path, matrix, form, rows, cols, per, lam, epochs=0, warm=0):
    return dict(path=path, matrix=matrix, form=form, rows=int(rows), cols=int(cols), per=int(per), lam=float(lam),
                epochs=epochs, warm=warm)


def listed():
    return [
        # The smallest fit: 200 dense features, milliseconds in all, where launches and latency count.
        dict(_case("train", "dense", "ridge_primal", 2_000, 200, 200, 1e-3, epochs=16), name="dense_fit"),
        # The sparse regression workload with its strong regularisation: nothing limits the concurrency.
        dict(_case("train", "uniform", "ridge_primal", 100_000, 50_000, 50, 1e-2, epochs=4), name="sparse_fit"),
        # The same regression weakly regularised, as at the end of a regularisation path: hundreds in flight.
        dict(_case("train", "uniform", "ridge_primal", 100_000, 50_000, 50, 1e-5, epochs=30), name="sparse_weak_fit"),
        # The dual form of it, over examples.
        dict(_case("train", "uniform", "ridge_dual", 100_000, 50_000, 50, 1e-4, epochs=16), name="sparse_dual_fit"),
        # A text classifier on a small corpus.
        dict(_case("train", "text", "svm_dual", 3_500, 166_000, 370, 1 / 3_500, epochs=12), name="text_small_fit"),
        # An epoch of the text classifier on the full corpus, 1.3 billion entries, with its convergence check.
        dict(_case("resume", "text", "svm_dual", 350_000, 16_600_000, 3_700, 1 / 350_000, epochs=1, warm=10),
             name="text_large"),
        # The same corpus by terms: columns of one to 350,000 entries.
        dict(_case("resume", "text", "ridge_primal", 350_000, 16_600_000, 3_700, 1 / 350_000, epochs=1, warm=8),
             name="terms_large"),
        # Click prediction on a small sample, a few epochs at a time.
        dict(_case("resume", "click", "svm_dual", 50_000, 75_000, FIELDS, 1 / 50_000, epochs=4, warm=24),
             name="click_small"),
        # Click prediction on a day's sample.
        dict(_case("resume", "click", "svm_dual", 2_000_000, 3_000_000, FIELDS, 10 / 2_000_000, epochs=1, warm=24),
             name="click_sample"),
        # An epoch of the full click log, 1.95 billion entries; regularised more strongly than 1/N, so that a
        # few epochs make a checkpoint from which two runs stay together.
        dict(_case("resume", "click", "svm_dual", 50_000_000, 75_000_000, FIELDS, 1000 / 50_000_000, epochs=1, warm=7),
             name="click_large"),
        # Predictions for 5 million examples.
        dict(_case("score", "click", "svm_dual", 5_000_000, 7_500_000, FIELDS, 1 / 5_000_000), name="click_score"),
        # What every fit begins with.
        dict(_case("create", "click", "svm_dual", 5_000_000, 7_500_000, FIELDS, 1 / 5_000_000), name="click_create"),
    ]


def draw(rng):
    def log(lo, hi):
        return int(math.exp(rng.uniform(math.log(lo), math.log(hi))))

    what = rng.choice(("dense", "sparse", "weak", "dual", "text", "text", "terms", "click", "click", "score", "create"))
    if what == "dense":
        rows = log(500, 8_000)
        return _case("train", "dense", "ridge_primal", rows, log(40, rows // 8), 0, 1e-3, epochs=16)
    if what in ("sparse", "weak", "dual"):
        rows = log(20_000, 300_000)
        cols, per = int(rows * rng.uniform(0.3, 0.9)), log(10, 100)
        if what == "dual":
            return _case("train", "uniform", "ridge_dual", rows, cols, per, 10 / rows, epochs=16)
        lam, epochs = (1e-2, 4) if what == "sparse" else (1 / rows, 30)
        return _case("train", "uniform", "ridge_primal", rows, cols, per, lam, epochs=epochs)
    if what in ("text", "terms"):
        rows, per = log(2_000, 100_000), log(200, 2_500)
        form = "svm_dual" if what == "text" else "ridge_primal"
        path, epochs, warm = ("train", 12, 0) if rows * per < 3_000_000 else ("resume", 1, 14)
        return _case(path, "text", form, rows, int(rows * rng.uniform(20, 50)) + 40 * per, per, 1 / rows, epochs, warm)
    rows = log(20_000, 3_000_000)
    cols = int(rows * rng.uniform(1.0, 1.6))
    if what == "click":
        return _case("resume", "click", "svm_dual", rows, cols, FIELDS, 10 / rows, epochs=2, warm=24)
    if rng.random() < 0.5:
        rows, per = log(2_000, 60_000), log(200, 2_500)
        return _case(what, "text", "svm_dual", rows, 40 * rows + 40 * per, per, 1 / rows)
    return _case(what, "click", "svm_dual", rows, cols, FIELDS, 1 / rows)


# --------------------------------------------------------------------------- the calls


def prepare(case, seed):
    matrix = _matrix(case, seed)
    torch.cuda.empty_cache()  # the library allocates its own memory
    state = {"case": case, "matrix": matrix}
    if case["path"] == "create":
        return state
    s = state["solver"] = scd.Solver(*matrix, case["lam"], case["form"])
    if case["path"] == "score":
        state["vector"] = torch.randn(s.L, device="cuda", generator=_generator(seed + 1))
        return state
    if case["warm"]:
        if s.info()["auto_window"] > 16 and case["matrix"] == "click":
            s.set_option("window", 16)
        s.epochs(EPOCH_SEED, case["warm"])
        s.set_option("window", 0)
    state["checkpoint"] = s.get_state()
    return state


def run(state):
    case = state["case"]
    if case["path"] == "create":
        with scd.Solver(*state["matrix"], case["lam"], case["form"]) as s:
            return {"norms": s.norms(), "coupling": s.info()["coupling"]}
    s = state["solver"]
    if case["path"] == "score":
        return {"scores": s.gather_dots(state["vector"])}
    s.set_state(*state["checkpoint"])
    s.epochs(EPOCH_SEED, case["epochs"])
    primal, dual = s.objective()
    model, shared, _ = s.get_state()
    return {"model": model, "shared": shared, "primal": primal, "dual": dual}


def _entries(case):
    return case["rows"] * (case["cols"] if case["matrix"] == "dense" else case["per"])


def work(case):
    n, path = _entries(case), case["path"]
    segs, length = case["rows"], case["cols"]
    if case["form"] == "ridge_primal":
        segs, length = length, segs
    a = 8 * n + 8 * segs  # the matrix, read once
    if path == "score":
        return {"bytes": a + 4 * length + 4 * segs, "flops": 2 * n}
    if path == "create":
        # read once to check it and to take its norms; the coupling estimate applies it and its
        # transpose to one vector at least
        return {"bytes": 3 * a + 8 * segs + 8 * length, "flops": 6 * n}
    # an epoch reads the matrix once, gathers and updates an entry of the shared vector for each of
    # its own; the objectives read it once more
    per_epoch = 16 * n + 24 * segs
    return {"bytes": case["epochs"] * per_epoch + a + 4 * n + 12 * segs + 12 * length,
            "flops": case["epochs"] * 4 * n + 2 * n}


def tolerance(case):
    if case["path"] == "score":
        return {"rel": 1e-5, "max": 1e-4}  # fp32 sums of 39 to 2,500 products
    if case["path"] == "create":
        return {"rel": 1e-4, "max": 1e-3}  # the coupling: a largest value of squared fp32 sums
    # Epochs are asynchronous: two runs of one state visit in the same order and read other coordinates'
    # updates at other times.  Stated: about four times what two runs differ by.
    if case["matrix"] in ("dense", "uniform"):
        return {"rel": 1e-5, "max": 2e-4}  # run to the minimiser
    if case["matrix"] == "click":
        return {"rel": 0.03, "max": 0.99} if case["rows"] < 10_000_000 else {"rel": 0.02, "max": 0.99}
    return {"rel": 0.02, "max": 0.99} if case["path"] == "resume" else {"rel": 5e-3, "max": 0.2}


# --------------------------------------------------------------------------- in 64 bits


def exact(case, seed):
    if _entries(case) > 400_000_000:
        return None
    rows, cols, ptr, idx, val, y = _matrix(case, seed)
    n_seg = ptr.numel() - 1
    length = rows if case["form"] == "ridge_primal" else cols
    v, at = val.double(), idx.long()
    seg = torch.repeat_interleave(torch.arange(n_seg, device="cuda"), ptr[1:] - ptr[:-1])

    def dots(u):  # of every segment with u
        return torch.zeros(n_seg, dtype=torch.float64, device="cuda").index_add_(0, seg, v * u[at])

    def spread(x):  # the transpose
        return torch.zeros(length, dtype=torch.float64, device="cuda").index_add_(0, at, v * x[seg])

    if case["path"] == "score":
        return {"scores": dots(torch.randn(length, device="cuda", generator=_generator(seed + 1)).double())}
    if case["path"] == "create":
        norms = torch.zeros(n_seg, dtype=torch.float64, device="cuda").index_add_(0, seg, v * v)
        return {"norms": norms, "coupling": None}
    if case["path"] != "train" or case["matrix"] == "text":
        return None
    # The minimiser, by conjugate gradients: of the primal (A^T A + N lam I) x = A^T y, of the dual
    # (A A^T + N lam I) x = lam y; at it both objectives have one value.
    lam, y = case["lam"], y.double()
    primal = case["form"] == "ridge_primal"
    r = dots(y) if primal else lam * y
    x, p, rr = torch.zeros_like(r), r.clone(), float(r @ r)
    stop = rr * 1e-30
    for _ in range(500):
        if rr <= stop:
            break
        q = dots(spread(p)) + rows * lam * p
        step = rr / float(p @ q)
        x += step * p
        r -= step * q
        rr, last = float(r @ r), rr
        p = r + (rr / last) * p
    w = spread(x)
    if primal:
        best = float((w - y).square().sum()) / (2 * rows) + lam / 2 * float(x @ x)
    else:
        best = float(y @ x) - rows / 2 * float(x @ x) - float(w @ w) / (2 * lam)
    return {"model": x, "shared": w, "primal": best, "dual": best}
