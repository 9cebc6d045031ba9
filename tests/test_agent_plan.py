"""The plans of agent-resident calls (host only): the models of
test_gpu_resident.py and test_gpu_agent_tile.py reach the kernels and forms
that those files say they test."""
import numpy as np
import pytest

from paper_2607_17855_amd import synth
from agent_plan import plan_of
import test_gpu_agent_tile as tile
import test_gpu_resident as res

ALGOS = ("fpi", "vmp", "mmp")


@pytest.mark.parametrize("form", range(len(res.FORMS)))
def test_resident_forms(form):
    n, U, deps, lists, T, fpi, vmp, *mmp = res.FORMS[form]
    w, _ = res.form_workload(form)
    kind = "coupled" if lists else "resident"
    for algo, text in zip(ALGOS, (fpi, vmp, mmp[0] if mmp else vmp)):
        p = plan_of(w.model, w.b, w.T, algo)
        assert p["kernel"] == res.kernel_of(kind, algo), p
        assert (p["tile"] if algo == "fpi" else f"{p['tile']} {p['tables']} {p['passes']}") == text, p


def test_every_kernel_has_a_form():
    tiles = {"1x1", "2x1", "4x1", "8x1", "2x2", "4x2", "8x2", "4x4", "6x4", "12x2", "8x4", "12x4", "12x5", "8x8"}
    passes = {"one", "several"}
    for algo in (0, 1):
        plain = [(f[6:] * 2)[algo].split() for f in res.FORMS if not f[3]]
        coupled = [(f[6:] * 2)[algo].split() for f in res.FORMS if f[3]]
        assert {(t, p) for t, _, p in plain} == {(t, p) for t in tiles - {"12x2"} for p in passes}   # (the filter's alone)
        assert {(b, p) for _, b, p in plain} == {(b, p) for b in ("twice", "once", "packed") for p in passes}
        assert {tuple(c) for c in coupled} == (
            {(t, "lds", p) for t in ("1x1", "2x2", "4x2", "4x4", "6x4", "12x4", "12x5") for p in passes}
            | {(t, "packed", p) for t in ("2x2", "4x2", "12x4") for p in passes})
    assert {f[5] for f in res.FORMS if not f[3]} == tiles


@pytest.mark.parametrize("algo", ALGOS)
def test_resident_cases(algo):
    for kind, names, make in (("resident", res.CASES, res._workload), ("streamed", res.STREAMED, res._workload),
                              ("coupled", res.COUPLED, res._coupled)):
        if algo == "fpi" and kind == "streamed":
            continue
        for name in names:
            w, _ = make(name)
            p = plan_of(w.model, w.b, w.T, algo)
            assert p["kernel"] == res.kernel_of(kind, algo, w.T), (name, p)
    w, _ = res._coupled("long_lists")
    assert plan_of(w.model, w.b, w.T, "fpi")["kernel"] == "agent_filter_resident"


@pytest.mark.parametrize("algo", ("vmp", "mmp"))
def test_streamed_cases(algo):
    """The three places of the tables; windows at once and in chunks; both
    orders of the walk (flipped: lists of four with the closer states divided
    among the lanes)."""
    plans = []
    for name in res.STREAMED:
        w, _ = res._workload(name)
        plans.append((w.T, plan_of(w.model, w.b, w.T, algo)))
    assert {p["tables"] for _, p in plans} == {"twice", "once", "packed"}
    assert {int(p["chunk"]) < T for T, p in plans} == {True, False}
    assert {int(p["steps"]) < T for T, p in plans} == {True, False}
    flips = {n: int(p["flip"]) for n, (_, p) in zip(res.STREAMED, plans)}
    assert {n for n in flips if flips[n]} == {"rank4_three_columns", "five_columns", "flipped_walk"}


@pytest.mark.parametrize("algo", ("vmp", "mmp"))
def test_small_windows_of_many_lists(algo):
    """More than four maximal lists in a window that fits LDS: streamed while
    all workgroups (8 waves to a compute unit) run at once, else staged; a
    window that does not fit LDS is streamed for any number of agents."""
    small = _model([3, 4, 2, 3, 4, 2], [2, 1, 2, 1, 1, 1], [4] * 5, [[0, 1], [1, 2], [2, 3], [3, 4], [4, 5]])
    waves = int(plan_of(small, 1, 9, algo)["threads"]) // 64
    assert 2 <= waves <= 4
    fit = 8 // waves * 256
    for b in (1, 256, fit):
        assert plan_of(small, b, 9, algo)["kernel"] == "agent_window_streamed"
    for b in (fit + 1, 2048, 100000):
        assert plan_of(small, b, 9, algo)["kernel"] == "agent_window"
    large = _model([20, 18, 16, 3, 4, 2], [2, 1, 2, 1, 1, 1], [4] * 5, [[0, 1], [1, 2], [2, 3], [3, 4], [4, 5]])
    for b in (1, 2048):
        assert plan_of(large, b, 20, algo)["kernel"] == "agent_window_streamed"


def _model(n, U, K, deps):
    return synth.make_model(np.random.Generator(np.random.PCG64(1)), n, U, K, deps, 1, 1.0, 1.0)


def test_tile_cases():
    for (n, U, K, deps, b, T, _), kernel in zip(tile.CASES, tile.KERNEL):
        for algo in ("vmp", "mmp"):
            assert plan_of(_model(n, U, K, deps), b, T, algo)["kernel"] == kernel
    for (n, K, deps, b, T), (fpi, window) in zip(tile.FPI_CASES, tile.FPI_KERNEL):
        for algo in ALGOS:
            assert plan_of(_model(n, [2] * len(n), K, deps), b, T, algo)["kernel"] == (fpi if algo == "fpi" else window)
    for n, U, K, deps, b, T, *form in tile.FORMS.values():
        for algo in ALGOS:
            assert plan_of(_model(n, U, K, deps), b, T, algo).get("src", "") == form[algo != "fpi"]


def test_bench_knows_every_kernel():
    """The benchmark's record names the kernel of each profile class and its
    sources, and counts merged tensors once per maximal list."""
    import bench
    kernels = {"agent_window", "agent_window_tile", "agent_filter", "agent_filter_tile", "agent_filter_resident",
               "agent_window_resident", "agent_window_coupled", "agent_window_streamed"}
    assert set(bench.AGENT_KERNELS) == kernels
    for name, sources, _ in bench.AGENT_KERNELS.values():
        assert any(f" {name}(" in open(f"{bench.CSRC}/{s}").read() for s in sources)
    m = _model([2, 3, 5, 7], [1] * 4, [2] * 6, [[0], [0, 1], [0, 1], [1, 2], [3], [2]])
    assert sorted(bench.merged_sizes(m)) == [6, 7, 15]
