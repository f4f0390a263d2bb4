"""Policy search (Alg. 2, one frequency interval per pack) on the GPU through the C ABI, against
the search oracle (needs an MI355X).  Graphs whose energies lie on a dyadic grid keep every
makespan and energy exact in fp32, so both sides take every decision on the same numbers."""
import dataclasses
import json
import math
import os

import numpy as np
import pytest

import pins
from oracle import dp
from paper_2607_12324_amd import synth

pytestmark = pytest.mark.gpu
HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def torch():
    import torch as t
    assert t.cuda.is_available(), "GPU tests need a GPU"
    return t


@pytest.fixture(scope="module")
def emo(torch):
    from paper_2607_12324_amd import emo as mod
    return mod


def run(emo, gh, tgt, q, order=None, max_states=4096):
    lv, res = gh.dp_search(tgt, q, order, max_states=max_states)
    sel = emo.parse_selection(res)
    return lv.cpu().numpy(), sel


def check(emo, g, gh, tgt, q, order=None, what=""):
    r = dp.dp_search(g, tgt, q, order)
    lv, sel = run(emo, gh, tgt, q, order)
    assert sel.num_feasible == r.num_states, what
    if r.levels is None:
        assert sel.index == -1 and math.isnan(sel.energy) and math.isnan(sel.makespan), what
        return r
    assert np.array_equal(lv, r.levels), what
    assert sel.energy == r.energy and sel.makespan == r.makespan, what
    assert sel.index == math.floor(r.makespan / float(np.float32(q))), what
    return r


def test_dp_handworked(torch, emo):
    g = pins.graph_from_golden(pins.load_golden())
    gh = emo.EmoGraph(g, device=0)
    with open(os.path.join(HERE, "golden", "handworked_dp.json")) as f:
        cases = json.load(f)["cases"]
    for case in cases:
        print(f"[case] dp hand-worked {case['latency_target']} {case['quantum']} {case['pack_order']}", flush=True)
        lv, sel = run(emo, gh, case["latency_target"], case["quantum"], case["pack_order"])
        assert sel.num_feasible == case["num_states"], case
        if case["levels"] is None:
            assert sel.index == -1, case
        else:
            assert list(lv) == case["levels"], case
            assert sel.energy == case["energy"] and sel.makespan == case["makespan"], case


def dyadic(g, rng, step=2.0 ** -6):
    """The same graph with energies rounded to multiples of `step` and a dyadic static power."""
    e = (np.round(g.pack_energy / step) * step).astype(np.float32)
    return dataclasses.replace(g, pack_energy=e, static_power=float(rng.choice([0.0, 0.25, 0.5])))


@pytest.mark.parametrize("seed", range(3))
def test_dp_matches_oracle_on_random_dags(torch, emo, seed):
    rng = np.random.default_rng(800 + seed)
    found = 0
    for i in range(8):
        g = dyadic(synth.random_dag(rng, int(rng.integers(4, 14)), float(rng.uniform(0.15, 0.5)), 0.75,
                                    int(rng.integers(2, 6))), rng)
        if g.num_packs == 0:
            continue
        gh = emo.EmoGraph(g, device=0)
        T0 = float(dp.eval_batch(g, np.full((1, g.num_packs), g.num_levels - 1, np.uint8))[0][0])
        for tr in (0.9, 1.1, 1.4):
            tgt = float(np.float32(T0 * tr))
            q = float(rng.choice([0.25, 0.75, 1.0, 3.0]))
            order = rng.permutation(g.num_packs) if rng.random() < 0.5 else None
            print(f"[case] dp random seed={seed} #{i} P={g.num_packs} F={g.num_levels} target={tgt} q={q}", flush=True)
            r = check(emo, g, gh, tgt, q, order, f"{seed}/{i}/{tr}")
            found += r.levels is not None
        gh.close()
    assert found > 0


def test_dp_on_inference_graph(torch, emo):
    """The 64-pack inference graph (energies rounded to 2^-10) with about a hundred buckets:
    64 stages of up to ~800 candidates, against the oracle."""
    rng = np.random.default_rng(2)
    g = dyadic(synth.config_graph(2), rng, 2.0 ** -10)
    g = dataclasses.replace(g, static_power=0.25)
    gh = emo.EmoGraph(g, device=0)
    T0 = float(dp.eval_batch(g, np.full((1, g.num_packs), g.num_levels - 1, np.uint8))[0][0])
    tgt = float(np.float32(1.05 * T0))
    q = 2.0 ** math.floor(math.log2(0.05 * T0 / 100))
    print(f"[case] dp inference graph T0={T0} target={tgt} q={q}", flush=True)
    r = check(emo, g, gh, tgt, q, None, "inference graph")
    assert r.levels is not None and r.num_states > 10


def test_dp_without_packs_and_argument_errors(torch, emo):
    z = np.zeros(0, np.int32)
    g = synth.Graph("fixed-only", 2, np.asarray([0], np.int32), np.asarray([1], np.int32),
                    np.asarray([-1, -1], np.int32), np.asarray([3.0, 4.5], np.float32), 0, 2,
                    np.zeros((0, 2), np.float32), np.zeros((0, 2), np.float32), 0.5)
    gh = emo.EmoGraph(g, device=0)
    lv, sel = run(emo, gh, 8.0, 1.0)
    assert sel.index == 7 and sel.makespan == 7.5 and sel.energy == 3.75 and sel.num_feasible == 1
    lv, sel = run(emo, gh, 7.0, 1.0)
    assert sel.index == -1 and sel.num_feasible == 0
    del z
    g = pins.graph_from_golden(pins.load_golden())
    gh = emo.EmoGraph(g, device=0)
    for kw, status in ((dict(latency_target=float("nan"), quantum=1.0), 1),
                       (dict(latency_target=20.0, quantum=0.0), 1),
                       (dict(latency_target=20.0, quantum=1.0, pack_order=[0, 0, 1]), 1),
                       (dict(latency_target=20.0, quantum=2.0 ** -10, max_states=8), 1)):
        with pytest.raises(emo.EmoError) as ei:
            gh.dp_search(**kw)
        assert ei.value.status == status, kw
    # the same search twice: the scratch is reused and the result repeats exactly
    a = run(emo, gh, 20.0, 1.0)
    b = run(emo, gh, 20.0, 1.0)
    assert np.array_equal(a[0], b[0]) and a[1] == b[1]


@pytest.mark.parametrize("k", [2, 3])
def test_dp_on_workload_tables(torch, emo, k):
    """The search on the 64- and 512-pack workload graphs with their own (non-dyadic) energies,
    64 buckets between T0 and 1.05 T0.  Energies in fp32 can tie differently on the two sides
    and lead the searches through different stored policies, so the result is accepted when it
    is feasible, evaluates (oracle) to the makespan and energy it reports, and its energy is
    within 1e-5 of the oracle search's best."""
    g = synth.config_graph(k)
    gh = emo.EmoGraph(g, device=0)
    P, F = g.num_packs, g.num_levels
    T0 = float(dp.eval_batch(g, np.full((1, P), F - 1, np.uint8))[0][0])
    tgt = float(np.float32(1.05 * T0))
    q = float(np.float32(0.05 * T0 / 64))
    print(f"[case] dp on workload {k} tables: P={P} F={F} target={tgt} q={q}", flush=True)
    r = dp.dp_search(g, tgt, q)
    lv, sel = run(emo, gh, tgt, q)
    assert r.levels is not None and sel.index >= 0
    assert sel.makespan <= tgt
    T, E = dp.eval_batch(g, lv[None, :])
    assert float(np.float32(T[0])) == sel.makespan
    assert abs(sel.energy - E[0]) <= 1e-5 * E[0]
    assert abs(sel.energy - r.energy) <= 1e-5 * r.energy, (sel.energy, r.energy)
    assert sel.index == math.floor(sel.makespan / float(np.float32(q)))
    print(f"  energy {sel.energy} vs oracle {r.energy}; states {sel.num_feasible} vs {r.num_states}", flush=True)


def _search_graph(kind):
    rng = np.random.default_rng(77)
    if kind == "training":                       # one-kernel evaluators, 512 packs
        return synth.config_graph(3)
    if kind == "odd-blocks":                     # a last energy block of 3 packs, 11 levels
        return synth.packed_graph(5, 131, 3, 11, sync_every=50)
    if kind == "segmented":                      # a table past one kernel's LDS, no cuts
        return synth.without_cuts(synth.packed_graph(6, 640, 4, 16))
    if kind == "cuts":                           # cut-segment evaluators, whole energy blocks
        return synth.packed_graph(7, 768, 3, 16)
    if kind == "cuts-ragged":                    # segments of 160 packs: blocks of 64, 64 and 32
        return dyadic(synth.packed_graph(8, 960, 5, 16, sync_every=160), rng)
    if kind == "one-level":
        return synth.packed_graph(9, 70, 2, 1)
    if kind == "wide-levels":
        return synth.stream_graph(10, 40, 2, 256)
    # fixed nodes between packs, several predecessors, nodes without successors
    return dyadic(synth.random_dag(rng, 60, 0.08, 0.6, 5, shuffle_ids=False, shuffle_packs=False), rng)


@pytest.mark.parametrize("kind", ["training", "odd-blocks", "segmented", "cuts", "cuts-ragged", "one-level",
                                  "wide-levels", "fixed-nodes"])
def test_dp_one_kernel_matches_stages(torch, emo, kind):
    """The one-kernel search (packs in visiting order, exact time sums) gives the search by stages
    (interpreted mode) bit for bit: levels, energy, makespan, bucket and state count, from one bucket
    to as many as one workgroup takes, including no feasible policy; past that, and off the grid or in
    another order, the search by stages runs."""
    g = _search_graph(kind)
    P, F = g.num_packs, g.num_levels
    ga, gi = emo.EmoGraph(g, device=0), emo.EmoGraph(g, device=0, kernel_mode=emo.KERNELS_INTERPRETED)
    T0 = float(dp.eval_batch(g, np.full((1, P), F - 1, np.uint8))[0][0])
    cases = [(1.05, 64), (1.0, 1), (1.3, 3), (0.5, 8), (1.02, 200 if F <= 16 else 20)]
    if kind == "training":   # (the fixed-node graph's 5 levels would pass the LDS limit first)
        cases += [(1.1, 16384 // F - 3), (1.1, 16384 // F + 40)]
    for ratio, nb in cases:
        tgt = float(np.float32(ratio * T0))
        q = float(np.float32(max(abs(ratio - 1.0), 0.01) * T0 / nb))
        print(f"[case] dp one kernel {kind} P={P} F={F} target={tgt} buckets~{nb}", flush=True)
        kw = dict(max_states=1 << 16)
        a, sa = run(emo, ga, tgt, q, **kw)
        one = ga.info()["last_kernels"] == 9
        b, sb = run(emo, gi, tgt, q, **kw)
        assert gi.info()["last_kernels"] == 0
        assert (sa.index, sa.num_feasible) == (sb.index, sb.num_feasible), (sa, sb)
        if sa.index >= 0:
            assert np.array_equal(a, b) and (sa.energy, sa.makespan) == (sb.energy, sb.makespan), (sa, sb)
        assert one == (ratio > 0.9 and nb * F < 16384), (ratio, nb, one)
    ga.dp_search(float(np.float32(1.05 * T0)), T0, np.arange(P)[::-1].copy())
    assert P == 1 or ga.info()["last_kernels"] != 9
    off = emo.EmoGraph(synth.scaled_times(g, 1.1), device=0)
    off.dp_search(float(np.float32(1.2 * T0)), T0)
    assert off.info()["last_kernels"] != 9


def _chains_with_fixed(S, P, n, F, seed):
    """P packs round-robin on S chains, n fixed nodes after each, and a last node that waits for all."""
    rng = np.random.default_rng(seed)
    src, dst, pack, dur, last = [], [], [], [], [-1] * S
    for p in range(P):
        for k in range(n + 1):
            pack.append(p if k == 0 else -1)
            dur.append(0.0 if k == 0 else float(rng.integers(1, 9)) / 4)
            v = len(pack) - 1
            if last[p % S] >= 0:
                src.append(last[p % S])
                dst.append(v)
            last[p % S] = v
    pack.append(-1)
    dur.append(1.0)
    src += last
    dst += [len(pack) - 1] * S
    t = np.sort(synth.quantize(rng.uniform(1, 9, (P, F))), axis=1)[:, ::-1].astype(np.float32).copy()
    return synth.Graph("chains-fixed", len(pack), np.asarray(src, np.int32), np.asarray(dst, np.int32),
                       np.asarray(pack, np.int32), np.asarray(dur, np.float32), P, F, t, (0.37 * t).astype(np.float32), 0.25)


@pytest.mark.parametrize("S, P, n, one", [(1, 12, 50, True), (1, 12, 150, False), (12, 24, 9, True), (12, 24, 40, False),
                                          (24, 24, 4, True), (24, 24, 18, False), (40, 40, 3, True), (40, 40, 12, False)])
def test_dp_with_many_fixed_nodes(torch, emo, S, P, n, one):
    """Fixed nodes after each pack cost the one-kernel search a chain of reads: past about the time of the
    launches they save, the search goes by stages; the results are interpreted mode's on both sides."""
    g = _chains_with_fixed(S, P, n, 8, 100 * S + n)
    ga, gi = emo.EmoGraph(g, device=0), emo.EmoGraph(g, device=0, kernel_mode=emo.KERNELS_INTERPRETED)
    T0 = float(dp.eval_batch(g, np.full((1, P), 7, np.uint8))[0][0])
    tgt, q = float(np.float32(1.2 * T0)), float(np.float32(0.2 * T0 / 30))
    print(f"[case] dp fixed nodes S={S} P={P} n={n} target={tgt}", flush=True)
    a, sa = run(emo, ga, tgt, q)
    assert (ga.info()["last_kernels"] == 9) == one
    b, sb = run(emo, gi, tgt, q)
    assert sa.index >= 0 and np.array_equal(a, b) and sa == sb
    ga.close()
    gi.close()


def test_dp_energy_on_ragged_cut_segments(torch, emo):
    """Cut-segment evaluators start their fp32 energy blocks anew at each segment: on segments of 160
    packs (blocks of 64, 64 and 32) with non-dyadic energies, whose sums round differently under any
    other split, the one-kernel search reports the found policy's evaluated energy and makespan."""
    g = synth.packed_graph(8, 960, 5, 16, sync_every=160)
    P, F = g.num_packs, g.num_levels
    gh = emo.EmoGraph(g, device=0)
    T0 = float(dp.eval_batch(g, np.full((1, P), F - 1, np.uint8))[0][0])
    plain = 0
    cases = [(r, nb) for r in (1.01, 1.02, 1.05, 1.1, 1.2, 1.3) for nb in (9, 64)]
    for ratio, nb in cases:
        tgt, q = float(np.float32(ratio * T0)), float(np.float32((ratio - 1.0) * T0 / nb))
        print(f"[case] dp ragged cut segments target={tgt} buckets~{nb}", flush=True)
        lv, res = gh.dp_search(tgt, q)
        assert gh.info()["last_kernels"] == 9
        sel = emo.parse_selection(res)
        T, E = gh.eval_policies(lv[None, :].contiguous())
        assert gh.info()["last_kernels"] == 5
        assert sel.index >= 0 and float(T[0]) == sel.makespan and float(E[0]) == sel.energy, (sel, T, E)
        # the same packs in blocks of 64 from the first one on: another fp32 sum
        e = g.pack_energy[np.arange(P), lv.cpu().numpy()]
        total = 0.0
        for k in range(0, P, 64):
            b = np.float32(0)
            for x in e[k:k + 64]:
                b = np.float32(b + x)
            total += float(b)
        plain += float(np.float32(total + g.static_power * sel.makespan)) == sel.energy
    assert plain < len(cases) - 3   # (the test can tell the splits apart)
    gh.close()


@pytest.mark.parametrize("kind", ["least-energy-zero", "wide-range", "zero-block"])
def test_dp_energies_that_could_round(torch, emo, kind):
    """The one-kernel search needs every fp64 sum of block sums to be exact: a block that may sum to
    zero, or block sums further apart than fp64 holds, take the search by stages, a block that is always
    zero does not; the results are those of interpreted mode either way."""
    g = synth.packed_graph(5, 131, 3, 11, sync_every=50)
    e = g.pack_energy.copy()
    if kind == "least-energy-zero":
        e[64:128, 0] = 0.0
    elif kind == "wide-range":
        e[:64] *= np.float32(2.0 ** -60)
    else:
        e[:64] = 0.0
    g = dataclasses.replace(g, pack_energy=e)
    P, F = g.num_packs, g.num_levels
    ga, gi = emo.EmoGraph(g, device=0), emo.EmoGraph(g, device=0, kernel_mode=emo.KERNELS_INTERPRETED)
    T0 = float(dp.eval_batch(g, np.full((1, P), F - 1, np.uint8))[0][0])
    tgt, q = float(np.float32(1.1 * T0)), float(np.float32(0.1 * T0 / 50))
    print(f"[case] dp energies {kind} target={tgt}", flush=True)
    a, sa = run(emo, ga, tgt, q)
    assert (ga.info()["last_kernels"] == 9) == (kind == "zero-block")
    b, sb = run(emo, gi, tgt, q)
    assert sa.index >= 0 and np.array_equal(a, b) and sa == sb
    ga.close()
    gi.close()


def test_dp_first_identity_search_under_capture(torch, emo):
    """A search captured into a graph after only searches in another order warmed its stream: the one-kernel
    search's program is not built during the capture (that allocates and copies), the captured search goes
    by stages, and the next search outside builds it; every replay gives the eager result."""
    g = synth.packed_graph(5, 131, 3, 11, sync_every=50)
    P, F = g.num_packs, g.num_levels
    T0 = float(dp.eval_batch(g, np.full((1, P), F - 1, np.uint8))[0][0])
    tgt, q = float(np.float32(1.1 * T0)), float(np.float32(0.1 * T0 / 50))
    gh = emo.EmoGraph(g, device=0)
    lv = torch.zeros(P, dtype=torch.uint8, device="cuda")
    res = torch.zeros(3, dtype=torch.int64, device="cuda")
    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    print("[case] dp capture after a search in another order", flush=True)
    with torch.cuda.stream(s):
        gh.dp_search(tgt, q, np.arange(P)[::-1].copy(), best_levels=lv, result=res)
    s.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=s):
        gh.dp_search(tgt, q, best_levels=lv, result=res)
    assert gh.info()["last_kernels"] != 9
    eager, sel = run(emo, gh, tgt, q)
    assert gh.info()["last_kernels"] == 9 and sel.index >= 0
    for _ in range(3):
        lv.zero_()
        res.zero_()
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert np.array_equal(lv.cpu().numpy(), eager) and emo.parse_selection(res) == sel
        run(emo, gh, tgt, 2 * q)   # the program's own eager work between replays
    del graph
    gh.close()
