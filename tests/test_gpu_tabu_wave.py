"""GPU parity of the one-wavefront-per-individual TabuCol tier (table
"wave8": byte gamma with a tabu flag in LDS, live tabu pairs in an LDS list)
against the CPU oracle (Section 2.7): every individual's best colouring,
f_best, iteration count, counters and trajectory fingerprint bit-identical.
Covers every row-width bucket of the scan (k up to 256), runs past the
2^15 wrap of the stored expiries, moves with more than 64 ties, scans of
several rounds, both give-up paths (a colour class passing 127 vertices,
the tabu list overflowing) with their 16-bit reruns, and the full
8192 x 100,000 run on G(500, 0.5) with 64 individuals replayed."""
import sys

import numpy as np
import pytest
import torch

import oracle
from small_graphs import complete, cycle, edgeless
from workloads import workload
from workloads.graphs import from_edges, gnp, planted_partite

pytestmark = pytest.mark.gpu


def say(*a):
    print(*a, flush=True)
    sys.stdout.flush()


@pytest.fixture(scope="module")
def dlm():
    import paper_2109_05948_amd as dlm
    return dlm


def gpu_run(dlm, g, starts, k, T, seed, ind_base=0, **kw):
    G = dlm.Graph.from_csr(g)
    col = torch.from_numpy(np.ascontiguousarray(starts, np.int16)).cuda()
    r = dlm.tabu_batch(G, col, k, T, seed, ind_base=ind_base, table="wave8", **kw)
    torch.cuda.synchronize()
    out = {kk: (v.cpu().numpy() if isinstance(v, torch.Tensor) else v) for kk, v in r.items()}
    if out.get("hash") is not None:
        out["hash"] = out["hash"].view(np.uint64)
    return out


def compare(gpu, ref, ids, label):
    for j, i in enumerate(ids):
        msg = f"{label} individual {i}"
        assert gpu["f_best"][j] == ref["f_best"][j], (msg, gpu["f_best"][j], ref["f_best"][j])
        assert gpu["iters"][j] == ref["iters"][j], (msg, gpu["iters"][j], ref["iters"][j])
        assert (gpu["stats"][j][:6] == ref["stats"][j][:6]).all(), (msg, gpu["stats"][j], ref["stats"][j])
        assert gpu["hash"][j] == ref["hash"][j], msg
        assert (gpu["colors"][j] == ref["colors"][j]).all(), msg


SHAPES = [  # (n, p, k, T, pop): row buckets of 8, 16, 24, 32 and 64 dwords, exact widths 9 to 15 and 17 to 23
    (37, 0.3, 4, 800, 7),
    (150, 0.5, 16, 3000, 9),
    (200, 0.1, 5, 3000, 5),
    (120, 0.9, 40, 2000, 6),
    (300, 0.5, 33, 2500, 4),
    (260, 0.8, 70, 2000, 4),
    (330, 0.9, 100, 1500, 3),
    (420, 0.95, 210, 800, 3),
    (160, 0.5, 44, 1500, 3),  # 11 dwords
    (140, 0.6, 47, 1500, 3),  # 12
    (180, 0.5, 55, 1500, 3),  # 14
    (200, 0.5, 58, 1200, 3),  # 15
    (220, 0.6, 67, 1000, 3),  # 17
    (240, 0.5, 75, 1000, 3),  # 19
    (200, 0.7, 79, 1000, 3),  # 20
    (260, 0.5, 83, 1000, 3),  # 21
    (250, 0.6, 90, 1000, 3),  # 23
    (300, 0.5, 96, 1000, 3),  # 24: the bucket at its own width
]


@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "n%d_p%g_k%d" % s[:3])
def test_wave_parity_shapes(dlm, dev, shape):
    n, p, k, T, pop = shape
    g = gnp(n, p, seed=n)
    starts = oracle.init_random(n, k, pop, seed=3, ind_base=11)
    ids = np.arange(11, 11 + pop)
    ref = oracle.tabucol_batch(g, starts, ids, k, T, seed=17)
    say(f"wave8 n={n} p={p} k={k} T={T} pop={pop}")
    gpu = gpu_run(dlm, g, starts, k, T, 17, ind_base=11)
    compare(gpu, ref, ids, f"wave8 n{n} k{k}")


def test_wave_long_run_past_expiry_wrap(dlm, dev):
    """40,000 iterations: the stored expiries (modulo 2^15) wrap."""
    g = gnp(120, 0.5, seed=7)
    k, T, pop = 13, 40000, 4
    starts = oracle.init_random(g.n, k, pop, seed=5)
    ref = oracle.tabucol_batch(g, starts, np.arange(pop), k, T, seed=8)
    assert (ref["iters"] == T).all()  # no individual stops early
    say(f"wave8 long run n=120 k={k} T={T}")
    gpu = gpu_run(dlm, g, starts, k, T, 8)
    compare(gpu, ref, range(pop), "wave8 long")


def test_wave_trace(dlm, dev):
    g = gnp(90, 0.5, seed=2)
    k, T = 11, 600
    starts = oracle.init_random(90, k, 3, seed=1)
    say("wave8 trace n=90 k=11")
    gpu = gpu_run(dlm, g, starts, k, T, 4, trace_cap=T)
    for i in range(3):
        ref = oracle.tabucol(g, starts[i], k, T, seed=4, ind=i, trace_cap=T)
        it = ref["iters"]
        assert (gpu["trace"][i][:it] == ref["trace"][:it]).all()


def test_wave_edge_cases(dlm, dev):
    cases = [
        ("edgeless", edgeless(40), 1, 50),
        ("K9 k=3", complete(9), 3, 400),
        ("K9 k=9", complete(9), 9, 400),
        ("C7 k=2", cycle(7), 2, 300),
        ("k=1", gnp(30, 0.2, seed=1), 1, 50),
        ("T=0", gnp(30, 0.2, seed=1), 3, 0),
        ("planted", planted_partite(200, 8, 0.5, seed=4)[0], 8, 4000),
    ]
    for name, g, k, T in cases:
        starts = oracle.init_random(g.n, k, 3, seed=2)
        ref = oracle.tabucol_batch(g, starts, np.arange(3), k, T, seed=6)
        say(f"wave8 edge case {name}")
        gpu = gpu_run(dlm, g, starts, k, T, 6)
        compare(gpu, ref, range(3), name)
    # an out-of-range start colour is refused per individual
    g = gnp(30, 0.3, seed=0)
    starts = oracle.init_random(g.n, 4, 2, seed=1)
    starts[1, 5] = 4
    gpu = gpu_run(dlm, g, starts, 4, 100, 1)
    assert gpu["f_best"][1] == -1 and gpu["iters"][1] == -1 and gpu["iters"][0] >= 0


def test_wave_many_ties(dlm, dev):
    """A perfect matching on 1000 vertices with k = 120: each conflicting
    vertex ties at delta -1 with every free colour, about 2,000 tied moves
    per iteration, so the ties are hashed 64 at a time."""
    n, k, T, pop = 1000, 120, 40, 3
    g = from_edges(n, np.array([(2 * i, 2 * i + 1) for i in range(n // 2)], np.int64), "matching1000")
    starts = oracle.init_random(n, k, pop, seed=9)
    ref = oracle.tabucol_batch(g, starts, np.arange(pop), k, T, seed=5)
    assert (ref["stats"][:, 4] > 0).all()
    say(f"wave8 matching1000 k={k}")
    gpu = gpu_run(dlm, g, starts, k, T, 5)
    compare(gpu, ref, range(pop), "wave8 matching")


def _class_sizes_over_run(start, k, trace, iters):
    col = start.astype(np.int64).copy()
    size = np.bincount(col, minlength=k)
    worst = [int(size.max())]
    for t in range(iters):
        rec = int(trace[t][0])
        if rec < 0:
            continue
        v, c = rec & 0xffff, rec >> 16
        size[col[v]] -= 1
        size[c] += 1
        col[v] = c
        worst.append(int(size.max()))
    return worst


def test_wave_reruns_when_a_class_passes_127(dlm, dev):
    """k = 3 on 370 vertices: classes of about 123.  Individuals whose start
    has a class above 127 and individuals whose class grows past 127 during
    the search both give up and are rerun with 16-bit gamma."""
    g = gnp(370, 0.02, seed=11)
    k, T, pop = 3, 1500, 16
    starts = oracle.init_random(g.n, k, pop, seed=21)
    ids = np.arange(pop)
    ref = oracle.tabucol_batch(g, starts, ids, k, T, seed=5)
    at_start, mid_run = 0, 0
    for i in range(pop):
        tr = oracle.tabucol(g, starts[i], k, T, seed=5, ind=i, trace_cap=T)
        worst = _class_sizes_over_run(starts[i], k, tr["trace"], tr["iters"])
        at_start += worst[0] > 127
        mid_run += worst[0] <= 127 and max(worst) > 127
    assert at_start > 0 and mid_run > 0, (at_start, mid_run)
    say(f"wave8 rerun n=370 k=3 ({at_start} at start, {mid_run} mid-run)")
    gpu = gpu_run(dlm, g, starts, k, T, 5)
    compare(gpu, ref, ids, "wave8 class rerun")


def test_wave_reruns_when_the_tabu_list_overflows(dlm, dev):
    """G(2000, 0.9) with k = 64: f stays above 20,000, so every tenure
    exceeds 12,000 iterations and each of the 8,000 moves leaves a live tabu
    pair.  The table fills 139 KB of the 160 KB LDS, leaving room for about
    6,000 pairs: the list overflows, the individual gives up and its 16-bit
    rerun must still equal the oracle."""
    g = gnp(2000, 0.9, seed=3)
    k, T, pop = 64, 8000, 2
    starts = oracle.init_random(g.n, k, pop, seed=4)
    ref = oracle.tabucol_batch(g, starts, np.arange(pop), k, T, seed=6)
    assert (ref["f_best"] > 20000).all() and (ref["stats"][:, 0] > 7800).all()
    say("wave8 tabu-list overflow n=2000 k=64")
    gpu = gpu_run(dlm, g, starts, k, T, 6)
    compare(gpu, ref, range(pop), "wave8 list overflow")


def test_wave_gnp1000_k85(dlm, dev):
    """G(1000, 0.5), k = 85 (the memetic shape): scans of several rounds."""
    g = gnp(1000, 0.5, seed=0)
    k, T, pop = 85, 4000, 6
    starts = oracle.init_random(g.n, k, pop, seed=3)
    ref = oracle.tabucol_batch(g, starts, np.arange(pop), k, T, seed=9)
    say("wave8 gnp1000 k=85")
    gpu = gpu_run(dlm, g, starts, k, T, 9)
    compare(gpu, ref, range(pop), "wave8 gnp1000")


def test_wave_gnp500_full_size_sampled(dlm, dev):
    """G(500, 0.5), k = 49, 8192 individuals x 100,000 iterations in one
    wave8 launch; individuals i = 128 j replayed by the oracle, and for
    every individual f_best = conflicts of the returned colouring."""
    w = workload("gnp500")
    g, k, T = w.graphs[0], w.k[0], w.iters[0]
    G = dlm.Graph.from_csr(g)
    col, _ = dlm.init_population(G, k, w.pop, seed=w.init_seed)
    starts = col.cpu().numpy()
    say("wave8 gnp500 full size: 8192 x 100000")
    r = dlm.tabu_batch(G, col, k, T, w.tabu_seed, table="wave8")
    torch.cuda.synchronize()
    ids = np.arange(0, w.pop, w.extra["sample_stride"])
    ref = oracle.tabucol_batch(g, starts[ids], ids, k, T, seed=w.tabu_seed)
    gpu = {kk: v.cpu().numpy()[ids] for kk, v in r.items() if isinstance(v, torch.Tensor)}
    gpu["hash"] = gpu["hash"].view(np.uint64)
    compare(gpu, ref, ids, "wave8 gnp500")
    fb = r["f_best"].cpu().numpy()
    conf, _ = dlm.evaluate(G, r["colors"], k)
    assert (conf.cpu().numpy() == fb).all()
    st = r["stats"].cpu().numpy()
    assert (st[:, 0] + st[:, 1] == r["iters"].cpu().numpy()).all()


def test_wave_static_entry_point(dlm, dev):
    """The allocation-free entry point runs the wave tier too."""
    g = gnp(150, 0.5, seed=3)
    k, T, pop = 16, 3000, 9
    G = dlm.Graph.from_csr(g)
    starts = oracle.init_random(g.n, k, pop, seed=2)
    ref = oracle.tabucol_batch(g, starts, np.arange(pop), k, T, seed=5)
    col = torch.from_numpy(starts.copy()).cuda()
    out = {"f_best": torch.empty(pop, dtype=torch.int32, device="cuda"),
           "iters": torch.empty(pop, dtype=torch.int32, device="cuda"),
           "stats": torch.empty((pop, 8), dtype=torch.int64, device="cuda"),
           "hash": torch.empty(pop, dtype=torch.int64, device="cuda")}
    say("wave8 static entry point")
    r = dlm.tabu_batch_static(G, col, k, T, 5, out, table="wave8")
    torch.cuda.synchronize()
    gpu = {kk: v.cpu().numpy() for kk, v in r.items()}
    gpu["hash"] = gpu["hash"].view(np.uint64)
    compare(gpu, ref, range(pop), "wave8 static")


WIDTHS = [  # (n, p, k, T, pop, sampled rows): entry width, waves per individual, row dwords
    (100, 0.5, 9, 2000, 4, None),            # 4 bits, one wave
    (300, 0.5, 22, 2000, 5, None),           # 4 bits, four waves, entries that outgrow 4 bits
    (340, 0.3, 18, 2000, 600, (0, 255, 599)),     # 4 bits, three individuals per CU
    (430, 0.5, 40, 500, 600, (0, 300, 599)),      # 4 bits, two waves
    (220, 0.5, 22, 300, 700, (0, 255, 699)),      # three individuals per CU, one wave each
    (600, 0.5, 44, 1500, 3, None),           # the same with four waves and more escapes than a register bank
    (400, 0.97, 256, 400, 3, None),          # 4 bits, 32 dwords, every 8-bit colour in use
    (1100, 0.6, 110, 300, 2, None),          # 4 bits, the 16-dword bucket, rows past 512 neighbours
    (1000, 0.95, 100, 400, 2, None),         # 8 bits, four waves, 25 dwords
    (520, 0.95, 250, 300, 3, None),          # 4 bits, 32 dwords
    (990, 0.99, 130, 200, 2, None),          # 8 bits, 33 dwords in the bucket of 64
    (300, 0.3, 14, 200, 6000, (0, 2999, 5999)),   # one wave above 256 vertices: the CU is full of individuals
    (600, 0.1, 12, 150, 2000, (0, 777, 1999)),    # two waves above 512 vertices
]


@pytest.mark.parametrize("shape", WIDTHS, ids=lambda s: "n%d_p%g_k%d" % s[:3])
def test_wave_entry_widths_and_waves(dlm, dev, shape):
    n, p, k, T, pop, rows = shape
    g = gnp(n, p, seed=n + k)
    starts = oracle.init_random(n, k, pop, seed=5, ind_base=3)
    at = np.arange(pop) if rows is None else np.array(rows)
    ref = oracle.tabucol_batch(g, starts[at], at + 3, k, T, seed=23)
    say(f"wave8 widths n={n} p={p} k={k} T={T} pop={pop}")
    gpu = gpu_run(dlm, g, starts, k, T, 23, ind_base=3)
    compare({x: gpu[x][at] for x in ("f_best", "iters", "stats", "hash", "colors")}, ref, at, f"widths n{n} k{k}")


def test_wave_reruns_when_many_entries_outgrow_four_bits_at_once(dlm, dev):
    """K(100, 100) with colours 0..6 on both sides, k = 20: the neighbours of a
    vertex share their rows, so a class of one side growing from 14 to 15
    makes 100 entries escape in one move, more than the 64 a move may hand
    over; the individual gives up and its rerun equals the oracle."""
    n, k, T, pop = 200, 20, 400, 4
    g = from_edges(n, np.array([(i, 100 + j) for i in range(100) for j in range(100)], np.int64), "K(100,100)")
    starts = oracle.init_random(n, 7, pop, seed=6)
    assert all(np.bincount(s[:100], minlength=7).max() >= 14 for s in starts)
    ref = oracle.tabucol_batch(g, starts, np.arange(pop), k, T, seed=7)
    say("wave8 mass escape K(100,100) k=20")
    gpu = gpu_run(dlm, g, starts, k, T, 7)
    compare(gpu, ref, range(pop), "mass escape")


def test_wave_reruns_when_the_side_list_overflows(dlm, dev):
    """All vertices in one class: f starts at every edge, far above a random
    start's, so tenures far exceed what the LDS share of one of 8192
    individuals was sized for."""
    n, k, T, pop = 120, 12, 500, 8192
    g = gnp(n, 0.5, seed=4)
    starts = np.zeros((pop, n), np.int16)
    at = np.array([0, 1, 4095, 8191])
    ref = oracle.tabucol_batch(g, starts[at], at, k, T, seed=3)
    say("wave8 side-list overflow n=120 k=12")
    gpu = gpu_run(dlm, g, starts, k, T, 3)
    compare({x: gpu[x][at] for x in ("f_best", "iters", "stats", "hash", "colors")}, ref, at, "side list")


def test_wave_table_beyond_two_to_the_seventeen(dlm, dev):
    """G(800, 0.9), k = 185: 148,800 entries, in 4 bits; the automatic table
    takes the wave tier, an explicit wave8 stays refused."""
    n, k, T, pop = 800, 185, 250, 2
    g = gnp(n, 0.9, seed=8)
    starts = oracle.init_random(n, k, pop, seed=2)
    ref = oracle.tabucol_batch(g, starts, np.arange(pop), k, T, seed=4)
    say("auto table n=800 k=185")
    G = dlm.Graph.from_csr(g)
    with pytest.raises(dlm.DlmError):
        dlm.tabu_batch(G, torch.from_numpy(starts).cuda(), k, T, 4, table="wave8")
    r = dlm.tabu_batch(G, torch.from_numpy(starts).cuda(), k, T, 4)
    torch.cuda.synchronize()
    gpu = {x: v.cpu().numpy() for x, v in r.items() if isinstance(v, torch.Tensor)}
    gpu["hash"] = gpu["hash"].view(np.uint64)
    compare(gpu, ref, range(pop), "large table")


@pytest.mark.parametrize("pop", [2, 3, 300, 600, 2000])
def test_wave_table_beyond_two_to_the_seventeen_asks_for_no_more_workspace(dlm, dev, pop):
    """Tables of that size went to device memory before: the start colourings
    and rerun slots of the wave table must not need more than that did."""
    n, k = 1000, 223
    G = dlm.Graph.from_csr(gnp(n, 0.9, seed=4))
    assert dlm.tabu_workspace_bytes(G, pop, k, 100) <= dlm.tabu_workspace_bytes(G, pop, k, 100, table="global16")


LONG = [  # (n, p, k, T, pop): 4 bits and one wave, four waves, 8 bits, a table beyond 2^17 entries
    (60, 0.5, 5, 3000, 3), (300, 0.5, 22, 2500, 2), (300, 0.95, 12, 2500, 2), (800, 0.9, 185, 4000, 2)]


@pytest.mark.parametrize("shape", LONG, ids=lambda s: "n%d_p%g_k%d" % s[:3])
def test_wave_tenures_past_two_to_the_fifteen(dlm, dev, shape):
    """ten_num = 32767, ten_den = 1 and ten_rand = 1024: the capped term of
    32,757 and the random term pass 2^15 together, so nearly every pair stays
    tabu to the end.  A stored expiry of 15 bits would free it within 1,012
    iterations of its move."""
    n, p, k, T, pop = shape
    g = gnp(n, p, seed=n + 1)
    starts = oracle.init_random(n, k, pop, seed=4)
    ten = {"ten_num": 32767, "ten_den": 1, "ten_rand": 1024}
    ref = oracle.tabucol_batch(g, starts, np.arange(pop), k, T, seed=12, **ten)
    assert (ref["f_best"] > 0).all()
    say(f"wave8 tenures past 2^15 n={n} k={k} T={T}")
    G = dlm.Graph.from_csr(g)
    table = "wave8" if n * k <= 1 << 17 else "auto"
    outs = [dlm.tabu_batch(G, torch.from_numpy(starts).cuda(), k, T, 12, table=table, **ten)]
    job = {"graph": G, "colors": torch.from_numpy(starts).cuda(), "k": k, "iters": T, "seed": 12, **ten}
    mb = dlm.MultiBatch([job])
    mb.launch()
    outs.append({**job, "iters": job["iters_out"]})
    torch.cuda.synchronize()
    for r, name in zip(outs, ("batch", "multi")):
        gpu = {x: r[x].cpu().numpy() for x in ("f_best", "iters", "stats", "hash", "colors")}
        gpu["hash"] = gpu["hash"].view(np.uint64)
        compare(gpu, ref, range(pop), f"long tenures {name} n{n} k{k}")


def test_wave_run_past_two_to_the_seventeen(dlm, dev):
    """140,000 iterations: the stored expiries (modulo 2^17) wrap, in the
    registers and, with the long tenures, in the LDS list."""
    g = gnp(60, 0.5, seed=9)
    k, T, pop = 6, 140000, 2
    starts = oracle.init_random(g.n, k, pop, seed=5)
    for ten in ({}, {"ten_num": 32767, "ten_den": 64, "ten_rand": 1024}):
        ref = oracle.tabucol_batch(g, starts, np.arange(pop), k, T, seed=8, **ten)
        assert (ref["iters"] == T).all()
        say(f"wave8 n=60 k={k} T={T} {ten}")
        gpu = gpu_run(dlm, g, starts, k, T, 8, **ten)
        compare(gpu, ref, range(pop), "wave8 2^17")


ROUTES = [  # (n, p, k, pop, T, tenure, 16-bit table in LDS): both sides of the line, by f, population, tenure, run length
    (480, 0.3, 6, 64, 300, {}, True), (480, 0.3, 21, 64, 300, {}, False),
    (300, 0.7, 12, 1024, 500, {}, True), (300, 0.7, 25, 1024, 300, {}, False), (300, 0.7, 25, 64, 300, {}, True),
    (100, 0.7, 5, 64, 400, {}, True), (100, 0.7, 5, 4096, 400, {}, False), (100, 0.7, 11, 64, 300, {}, False),
    (480, 0.3, 6, 64, 100, {}, False), (300, 0.5, 22, 3, 900, {"ten_num": 300}, True), (300, 0.5, 22, 3, 900, {}, False),
    (600, 0.02, 5, 3, 300, {}, True), (150, 0.1, 1, 3, 20, {}, True), (60, 0.1, 1, 3, 20, {}, False)]


@pytest.mark.parametrize("case", ROUTES, ids=lambda c: "n%d_p%g_k%d_pop%d" % c[:4])
def test_auto_table_where_many_pairs_are_tabu(dlm, dev, case):
    """The automatic table: the wave table refuses a call without workspace (it
    holds start colourings and rerun slots), the 16-bit table in LDS needs
    none; the workspace asked for is the same whatever the run's length."""
    n, p, k, pop, T, ten, lds16 = case
    g = gnp(n, p, seed=n)
    starts = oracle.init_random(n, k, pop, seed=6)
    at = np.unique([0, pop // 2, pop - 1])
    ref = oracle.tabucol_batch(g, starts[at], at, k, T, seed=3, **ten)
    G = dlm.Graph.from_csr(g)
    assert dlm.tabu_workspace_bytes(G, pop, k, T, **ten) == dlm.tabu_workspace_bytes(G, pop, k, 1, table="wave8")
    none = torch.empty(0, dtype=torch.uint8, device="cuda")
    if not lds16:
        with pytest.raises(dlm.DlmError):
            dlm.tabu_batch(G, torch.from_numpy(starts).cuda(), k, T, 3, workspace=none, **ten)
    say(f"auto table n={n} p={p} k={k} pop={pop} T={T} {ten}")
    r = dlm.tabu_batch(G, torch.from_numpy(starts).cuda(), k, T, 3, workspace=none if lds16 else None, **ten)
    torch.cuda.synchronize()
    gpu = {x: r[x].cpu().numpy()[at] for x in ("f_best", "iters", "stats", "hash", "colors")}
    gpu["hash"] = gpu["hash"].view(np.uint64)
    compare(gpu, ref, at, f"route n{n} k{k}")


@pytest.mark.parametrize("n,k,d,wave", [(5500, 40, 20, False), (4000, 45, 30, True)])
def test_auto_table_beyond_two_to_the_seventeen_by_class_size(dlm, dev, n, k, d, wave):
    """Tables that only 4-bit entries bring into the LDS: classes of 137
    vertices in the mean cannot stay within the wave table's 127, classes of
    89 can.  The device-memory table of two individuals asks for exactly
    their two tables, the wave table for one slot less and the starts."""
    g = gnp(n, d / n, seed=3)
    G = dlm.Graph.from_csr(g)
    T, pop = 150, 2
    auto, device = (dlm.tabu_workspace_bytes(G, pop, k, T, table=t) for t in ("auto", "global16"))
    assert (auto < device) == wave, (auto, device)
    starts = oracle.init_random(n, k, pop, seed=6)
    ref = oracle.tabucol_batch(g, starts, np.arange(pop), k, T, seed=3)
    say(f"auto table n={n} k={k} d={d}")
    r = dlm.tabu_batch(G, torch.from_numpy(starts).cuda(), k, T, 3)
    torch.cuda.synchronize()
    gpu = {x: r[x].cpu().numpy() for x in ("f_best", "iters", "stats", "hash", "colors")}
    gpu["hash"] = gpu["hash"].view(np.uint64)
    compare(gpu, ref, range(pop), f"large n{n} k{k}")


def star(n, leaves):
    """Vertex 0 joined to ``leaves`` others, which form a path."""
    e = [(0, v) for v in range(1, leaves + 1)] + [(v, v + 1) for v in range(1, leaves)]
    return from_edges(n, np.array(e, np.int64), f"star{n}")


def test_skewed_graph_takes_memory_by_its_entries(dlm, dev):
    """20,000 vertices, 80,000 entries, one row of 19,999: rows padded to the
    longest would take 800 MB."""
    g = star(20000, 19999)
    dlm.evaluate(dlm.Graph.from_csr(star(50, 40)), torch.zeros((1, 50), dtype=torch.int16, device="cuda"), 3)
    torch.cuda.synchronize()  # the library's kernels and fixed scratch are on the device from here on
    free = torch.cuda.mem_get_info()[0]
    G = dlm.Graph.from_csr(g)
    took = free - torch.cuda.mem_get_info()[0]
    say(f"star of 20,000: {took >> 10} KB")
    assert took < 16 << 20, took
    starts = oracle.init_random(g.n, 3, 2, seed=1)
    conf, _ = dlm.evaluate(G, torch.from_numpy(starts).cuda(), 3)
    ends = np.concatenate([[(0, v) for v in range(1, 20000)], [(v, v + 1) for v in range(1, 19999)]])
    assert (conf.cpu().numpy() == (starts[:, ends[:, 0]] == starts[:, ends[:, 1]]).sum(1)).all()


SKEWED = [  # (n, leaves, k, table): rows left out, with tables on both sides of 2^17 entries; rows kept
    (7000, 6999, 4, "wave8"), (7000, 6999, 4, "auto"), (5000, 4500, 50, "auto"), (4000, 3990, 32, "wave8")]


@pytest.mark.parametrize("case", SKEWED, ids=lambda c: "n%d_k%d_%s" % (c[0], c[2], c[3]))
def test_wave_on_skewed_graphs(dlm, dev, case):
    n, leaves, k, table = case
    g = star(n, leaves)
    T, pop = 300, 3
    starts = oracle.init_random(n, k, pop, seed=1)
    ref = oracle.tabucol_batch(g, starts, np.arange(pop), k, T, seed=2)
    bad = starts.copy()
    bad[1, n - 1] = k
    G = dlm.Graph.from_csr(g)
    say(f"star n={n} k={k} {table}")
    for rep in range(2):
        r = dlm.tabu_batch(G, torch.from_numpy(starts if rep == 0 else bad).cuda(), k, T, 2, table=table)
        torch.cuda.synchronize()
        gpu = {x: r[x].cpu().numpy() for x in ("f_best", "iters", "stats", "hash", "colors")}
        gpu["hash"] = gpu["hash"].view(np.uint64)
        at = np.array([0, 1, 2] if rep == 0 else [0, 2])
        compare({x: gpu[x][at] for x in gpu}, {x: ref[x][at] for x in ("f_best", "iters", "stats", "hash", "colors")},
                range(len(at)), f"star n{n} k{k}")
        if rep == 1:
            assert gpu["f_best"][1] == -1 and gpu["iters"][1] == -1
    job = {"graph": G, "colors": torch.from_numpy(starts).cuda(), "k": k, "iters": T, "seed": 2}
    mb = dlm.MultiBatch([job])
    mb.launch()
    torch.cuda.synchronize()
    assert (job["hash"].cpu().numpy().view(np.uint64) == ref["hash"]).all()


def groups(q, s, p, seed):
    """q groups of s vertices; two groups are joined completely with probability p."""
    rng = np.random.default_rng(seed)
    m = np.triu(rng.random((q, q)) < p, 1)
    lab = np.repeat(np.arange(q), s)
    e = np.argwhere(np.triu(m[np.ix_(lab, lab)] | m.T[np.ix_(lab, lab)], 1))
    return from_edges(q * s, e.astype(np.int64), f"groups{q}x{s}")


@pytest.mark.parametrize("q,s,p,k,pop", [(40, 20, 0.3, 40, 5), (16, 25, 0.3, 16, 40), (16, 25, 0.3, 16, 1500)])
def test_wave_reruns_with_bytes(dlm, dev, q, s, p, k, pop):
    """Groups of vertices with the same neighbours: a random start has few
    entries past 14, a good colouring thousands, so 4-bit entries give up on
    most individuals, whose rerun has 8-bit entries (and, for what these give
    up on, 16-bit ones); single calls and an uneven batch."""
    g = groups(q, s, p, seed=1)
    T = 500
    starts = oracle.init_random(g.n, k, pop, seed=2)
    at = np.unique(np.linspace(0, pop - 1, 40).astype(int))
    ref = oracle.tabucol_batch(g, starts[at], at, k, T, seed=7)
    say(f"wave8 groups {q}x{s} p={p} k={k} pop={pop}")
    gpu = gpu_run(dlm, g, starts, k, T, 7)
    compare({x: gpu[x][at] for x in ("f_best", "iters", "stats", "hash", "colors")}, ref, at, "groups")
    job = {"graph": dlm.Graph.from_csr(g), "colors": torch.from_numpy(starts).cuda(), "k": k, "iters": T, "seed": 7}
    other = gnp(150, 0.5, seed=1)
    st2 = oracle.init_random(150, 14, 6, seed=3)
    job2 = {"graph": dlm.Graph.from_csr(other), "colors": torch.from_numpy(st2).cuda(), "k": 14, "iters": 600, "seed": 8}
    ref2 = oracle.tabucol_batch(other, st2, np.arange(6), 14, 600, seed=8)
    mb = dlm.MultiBatch([job2, job])
    for rep in range(2):
        for j, st in ((job, starts), (job2, st2)):
            j["colors"].copy_(torch.from_numpy(st))
        mb.launch()
        torch.cuda.synchronize()
        for j, r, idx in ((job, ref, at), (job2, ref2, np.arange(6))):
            assert (j["hash"].cpu().numpy().view(np.uint64)[idx] == r["hash"]).all(), rep
            assert (j["iters_out"].cpu().numpy()[idx] == r["iters"]).all(), rep
            assert (j["colors"].cpu().numpy()[idx] == r["colors"]).all(), rep


def test_wave_reruns_when_a_conflict_list_is_full(dlm, dev):
    """Degrees of at most 16, so that every vertex that starts to conflict joins
    the list of the first of four waves (n / 2 + 64 entries); ten 4-cliques keep
    k = 3 conflicting, and tenures longer than the run force ever worse moves,
    until most of a colouring without other conflicts is in conflict."""
    n, k, d, T, pop = 330, 3, 16, 2000, 3
    rng = np.random.default_rng(1)
    deg, e = np.zeros(n, int), set()
    for q in rng.permutation(n)[:10 * (k + 1)].reshape(10, k + 1):
        for i in range(k + 1):
            for j in range(i):
                e.add((min(q[i], q[j]), max(q[i], q[j])))
                deg[q[i]] += 1
                deg[q[j]] += 1
    for a, b in rng.integers(0, n, (40 * n * d, 2)):
        if a % k != b % k and deg[a] < d and deg[b] < d and (min(a, b), max(a, b)) not in e:
            e.add((min(a, b), max(a, b)))
            deg[a] += 1
            deg[b] += 1
    g = from_edges(n, np.array(sorted(e), np.int64), "cliques")
    starts = np.tile((np.arange(n) % k).astype(np.int16), (pop, 1))
    ten = {"ten_num": 32767, "ten_den": 1, "ten_rand": 1024}
    for i in range(pop):  # conflicting vertices that began without a conflict, at the most
        tr = oracle.tabucol(g, starts[i], k, 400, seed=5, ind=i, trace_cap=400, **ten)
        col, most = starts[i].astype(int), 0
        ends = np.array(sorted(e))
        for rec in tr["trace"][:tr["iters"], 0]:
            if rec >= 0:
                col[rec & 0xffff] = rec >> 16
            bad = ends[col[ends[:, 0]] == col[ends[:, 1]]]
            most = max(most, len(np.unique(bad)))
        assert most - 10 * (k + 1) > n // 2, most
    ref = oracle.tabucol_batch(g, starts, np.arange(pop), k, T, seed=5, **ten)
    say("wave8 full conflict list")
    gpu = gpu_run(dlm, g, starts, k, T, 5, **ten)
    compare(gpu, ref, range(pop), "full list")
