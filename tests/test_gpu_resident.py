"""Register-resident agent kernels against the oracle, at the sizes where their
plan changes: every rank of a dependency list, one and several groups of
lists, a factor on no list, factors of one state, states on either side of a
tile's and a batch's edge, contexts side by side in a wave, factors spread
over several waves; with general B-dependency lists, lists of one and two
factors, with and without the factor itself, up to nine messages per state.
FORMS then names small models that reach every kernel built (tile shape, one
or several passes over the states, coupled tables in LDS and not) and every
place of the transition tables (in LDS twice, once, in the packed buffer);
test_agent_plan.py holds the plans of all these calls to what is said here.

All arithmetic is fp64 and the result fp32, so an output differs from the
fp64 oracle by its own rounding (3e-8 at most for a probability) and by what
the sweeps amplify of 1e-16: TOL leaves four roundings.
"""
import numpy as np
import pytest

from paper_2607_17855_amd import bi, synth
import oracle
from test_gpu_parity import check_invariants

pytestmark = pytest.mark.gpu
TOL = 1.2e-7

CASES = {
    # name: (n, U, K, deps, b, T, per_agent)
    "rank1": ([4], [2], [3], [[0]], 1, 8, False),
    "one_step": ([8, 6], [3, 1], [5, 7, 4], [[0, 1]] * 3, 9, 1, True),
    "rank2_edges": ([9, 5], [2, 3], [4, 3], [[0, 1], [1]], 5, 7, True),
    "rank3_subsets": ([12, 10, 8], [4, 2, 1], [6, 5, 4, 3], [[1], [0, 1], [0, 1, 2], [2]], 4, 20, True),
    "rank4": ([5, 3, 4, 2], [1, 2, 1, 3], [4, 3], [[0, 1, 2, 3], [1, 3]], 3, 6, False),
    "groups": ([7, 4, 6, 3], [2, 1, 2, 1], [5, 4, 3, 6], [[0, 1], [1, 2], [2, 3], [3]], 6, 5, False),
    "no_list": ([6, 5, 3], [2, 2, 2], [4], [[0, 2]], 4, 9, False),
    "one_state": ([1, 7, 1, 4], [1, 2, 1, 3], [3, 5], [[0, 1, 2, 3], [0, 2]], 5, 4, True),
    "long_factor": ([64, 3], [1, 2], [4, 3], [[0, 1], [0]], 3, 5, False),
    "chunks": ([33, 31, 30], [2, 1, 2], [3, 4], [[0, 1], [2]], 3, 4, False),
    "many_steps": ([5, 4], [3, 2], [4, 3], [[0, 1], [0]], 2, 90, True),
    "tables_several": ([26, 9], [5, 3], [3], [[1]], 3, 32, False),
    "tables_large": ([32, 31, 5], [5, 5, 2], [4], [[0]], 2, 17, False),
    "large_tile": ([22, 17, 9], [2, 1, 2], [4, 3], [[0, 1, 2], [0, 2]], 2, 3, False),
}

# general B-dependency lists: (n, U, K, deps, lists, b, T, per_agent)
COUPLED = {
    "pairs": ([12, 10, 8], [4, 2, 1], [6, 5, 4, 3], [[1], [0, 1], [0, 1, 2], [2]], [[0, 1], [1, 2], [0, 2]], 3, 20, True),
    "two_steps": ([5, 9], [2, 3], [4], [[0, 1]], [[0, 1], [0, 1]], 4, 2, False),
    "not_itself": ([4, 7, 3], [1, 2, 2], [3, 4], [[0, 2], [1]], [[1], [0, 2], [2]], 5, 11, True),
    # nine messages at factor 0 inside the window, one at the others
    "children": ([3, 2, 4, 2, 3, 2, 2, 5], [2, 1, 1, 2, 1, 1, 2, 1], [4, 3], [[0, 2], [1, 7]],
                 [[0]] + [[0, f] for f in range(1, 8)], 3, 5, False),
    "one_state": ([1, 6, 5], [1, 2, 1], [3], [[0, 1, 2]], [[0, 1], [0, 1], [1, 2]], 4, 6, True),
    "packed_tables": ([14, 13, 12], [5, 5, 4], [4], [[0, 1]], [[0, 1], [1, 2], [0, 2]], 2, 6, True),
    "many_steps": ([4, 5], [3, 2], [4, 3], [[0, 1], [0]], [[0, 1], [1]], 2, 70, True),
}
# (FPI takes lists of any length)
FILTER_LISTS = {"long_lists": ([4, 3, 2, 5], [1, 2, 2, 1], [3, 3], [[0, 1, 2, 3], [1, 3]],
                               [[0, 1, 2, 3], [0, 2, 3], [2], [1, 3]], 5, 7, True)}

# windows that exceed the registers: slices streamed in 4 x 4 blocks.  Rows of
# 1, 2, 3, 4 and 5 states, blocks that reach back, lists of one to four
# factors, all steps at once and in chunks, the tables' three places, several
# passes over the states
STREAMED = {
    "rank3": ([24, 21, 18], [2, 1, 2], [3, 2], [[0, 1, 2], [0, 2]], 3, 9, True),
    "rank4_two_columns": ([31, 11, 26, 2], [2, 1, 1, 2], [2, 3, 4], [[0, 1, 2, 3], [1, 3], [3]], 2, 5, False),
    "rank4_three_columns": ([17, 9, 13, 3], [1, 2, 1, 2], [2, 2, 3], [[0, 1, 2, 3], [3], [0, 2]], 2, 7, True),
    "one_column": ([30, 27, 25, 1], [2, 2, 1, 1], [3], [[0, 1, 2, 3]], 2, 4, False),
    "five_columns": ([32, 4, 21, 5], [1, 2, 2, 1], [2, 4], [[1, 2, 3], [0, 1, 2, 3]], 2, 6, False),
    "streamed_steps": ([25, 32], [3, 2], [3, 4], [[0, 1], [1]], 2, 28, True),
    "streamed_tables": ([32, 31, 30], [5, 5, 2], [2], [[0, 1, 2]], 2, 3, False),
    "streamed_no_list": ([6, 32, 31, 29], [2, 1, 1, 2], [2], [[1, 2]], 3, 24, False),
    # a list whose walk is flipped beside one without outer roles
    "flipped_walk": ([15, 32, 25, 6], [3, 2, 1, 2], [3, 2], [[0, 1, 2, 3], [1]], 2, 6, True),
}


# (n, U, deps, B-dependency lists or None, T, FPI's tile, the plan "tile tables
# passes" of VMP and, where it differs, of MMP), two agents with a model each
FORMS = [
    ([2], [1], [[0]], None, 2, "1x1", "1x1 twice one"),
    ([2, 4, 2], [2, 1, 4], [[0, 1, 2]], None, 2, "2x1", "2x1 twice one"),
    ([4, 3, 4], [2, 1, 1], [[0, 1, 2], [0, 1]], None, 2, "2x2", "2x2 twice one"),
    ([7, 2, 5], [1, 4, 1], [[0, 1, 2]], None, 2, "4x1", "4x1 twice one"),
    ([7, 9, 2], [1, 1, 5], [[0, 1, 2]], None, 2, "4x2", "4x2 twice one"),
    ([2, 13, 5, 3], [1, 1, 1, 2], [[0, 1, 2, 3], [0, 1]], None, 2, "8x2", "8x2 twice one"),
    ([3, 7, 3, 7], [2, 3, 1, 1], [[0, 2], [0, 1, 2, 3]], None, 2, "4x4", "4x4 twice one"),
    ([5, 5, 5, 4], [1, 4, 2, 4], [[0, 1, 2, 3], [1]], None, 2, "6x4", "6x4 twice one"),
    ([2, 3, 3, 13], [2, 1, 2, 3], [[0, 2], [0, 1, 2, 3]], None, 2, "8x1", "8x1 twice one"),
    ([3, 13, 7, 5], [4, 1, 1, 4], [[0, 2], [0, 1, 2, 3]], None, 2, "8x4", "8x4 twice one"),
    ([4, 4, 5, 17], [2, 2, 5, 1], [[0, 1, 2, 3]], None, 2, "12x2", "8x2 twice one"),
    ([3, 13, 4, 13], [5, 1, 3, 1], [[2]], None, 20, "1x1", "1x1 twice several"),
    ([3, 25, 5], [3, 1, 3], [[0, 2]], None, 20, "1x1", "8x1 twice several"),
    ([12, 17, 2, 2], [1, 2, 4, 1], [[0, 2]], None, 20, "2x1", "4x1 twice several"),
    ([4, 26, 4], [3, 1, 2], [[0, 2]], None, 20, "1x1", "4x4 twice several"),
    ([12, 2, 12, 7], [4, 1, 3, 3], [[1, 3]], None, 20, "1x1", "2x1 twice several"),
    ([5, 20, 5, 7], [2, 2, 3, 1], [[0, 1, 2, 3]], None, 2, "12x4", "12x4 twice one"),
    ([2, 9, 9, 20], [2, 5, 3, 1], [[2, 3], [0, 1, 2, 3]], None, 2, "12x5", "12x5 twice one"),
    ([5, 17, 2, 9], [1, 3, 3, 2], [[1, 2], [2, 3]], None, 32, "2x1", "4x2 twice several", "6x4 twice several"),
    ([13, 13, 3, 9], [4, 2, 5, 3], [[1, 3], [0, 1, 2, 3]], None, 2, "8x8", "8x8 twice one"),
    ([25, 9], [2, 4], [[0], [1]], None, 32, "1x1", "2x2 once several", "2x2 twice several"),
    ([9, 5, 25], [5, 4, 1], [[2], [0, 1]], None, 32, "2x1", "6x4 packed several", "4x2 once several"),
    ([2, 17, 13, 3], [1, 5, 2, 5], [[0, 2, 3], [0, 1]], None, 32, "4x1", "8x2 packed several"),
    ([33, 5], [1, 1], [[0, 1]], None, 32, "4x1", "12x5 once several", "12x5 twice several"),
    ([20, 9, 7], [2, 1, 5], [[0, 1], [2]], None, 32, "2x1", "8x4 once several", "8x4 twice several"),
    ([7, 4, 33], [1, 4, 1], [[1, 2]], None, 32, "4x1", "12x4 once several", "12x4 twice several"),
    ([5, 17, 5, 4], [1, 5, 4, 2], [[0, 3], [0, 1, 2]], None, 32, "4x1", "6x4 packed one"),
    ([13, 5, 9, 9], [2, 5, 2, 4], [[0, 1, 2]], None, 20, "4x2", "8x8 twice several"),
    ([7, 5, 13], [2, 1, 5], [[1], [0, 1, 2]], None, 32, "4x2", "6x4 once one"),
    ([2, 2], [1, 1], [[1], [1]], [[0], [0, 1]], 2, "1x1", "1x1 lds one"),
    ([4, 3, 2], [2, 1, 3], [[0, 1, 2], [0, 1, 2]], [[0], [1, 2], [2]], 2, "2x1", "2x2 lds one"),
    ([13, 5, 2], [1, 3, 2], [[0, 1, 2]], [[0], [1, 2], [2]], 2, "4x2", "4x2 lds one"),
    ([5, 4, 4, 5], [1, 3, 5, 5], [[0, 2], [0, 1, 2, 3]], [[0], [1, 3], [1, 2], [3]], 2, "4x4", "4x4 lds one"),
    ([5, 5, 5, 4], [5, 5, 2, 4], [[0, 1, 2, 3]], [[0], [1], [2, 3], [1, 3]], 2, "6x4", "6x4 lds one"),
    ([4, 2, 20, 7], [3, 1, 1, 1], [[3]], [[0], [0, 1], [2], [1, 3]], 20, "1x1", "2x2 lds several"),
    ([17, 4], [1, 2], [[1]], [[0], [0, 1]], 32, "1x1", "4x2 lds several"),
    ([20, 12, 2], [1, 3, 5], [[2]], [[0], [1], [1, 2]], 20, "1x1", "1x1 lds several"),
    ([13, 2, 20], [1, 1, 1], [[2]], [[0, 1], [1, 2], [2]], 20, "1x1", "2x2 packed several"),
    ([3, 3, 3, 9], [1, 3, 1, 4], [[0, 1, 3], [0, 2]], [[0], [1], [0, 2], [3]], 32, "4x1", "4x4 lds several"),
    ([5, 17], [1, 1], [[0]], [[0], [0, 1]], 32, "1x1", "2x2 packed one"),
    ([20, 13, 2], [1, 2, 1], [[0, 2]], [[0, 2], [1], [1, 2]], 20, "2x1", "4x2 packed several"),
    ([5, 7, 20, 5], [4, 1, 1, 1], [[0, 1, 2, 3]], [[0], [1], [2], [0, 3]], 2, "12x4", "12x4 lds one"),
    ([3, 9, 5], [5, 1, 3], [[0, 1, 2]], [[0], [0, 1], [2]], 32, "2x2", "6x4 lds several"),
    ([2, 5, 12, 17], [1, 4, 1, 1], [[0, 1, 2], [1, 3]], [[0, 3], [0, 1], [0, 2], [3]], 20, "4x1", "12x4 packed several"),
    ([5, 13, 9, 5], [1, 3, 2, 3], [[2, 3], [0, 1, 2, 3]], [[0, 3], [1], [2], [0, 3]], 3, "6x4", "12x5 lds one"),
    ([9, 13, 3], [3, 1, 2], [[0, 1, 2]], [[0, 2], [1], [1, 2]], 20, "4x2", "12x4 lds several"),
    ([5, 2, 7, 5], [1, 1, 1, 2], [[0, 1, 2, 3]], [[0], [1], [1, 2], [1, 3]], 32, "4x2", "12x5 lds several"),
    ([13, 13], [1, 2], [[0, 1]], [[0, 1], [0, 1]], 16, "1x1", "4x2 packed one"),
    ([20, 2, 9], [1, 5, 1], [[1], [0, 1, 2]], [[0, 2], [1], [0, 2]], 16, "4x2", "12x4 packed one"),
]


def _torch():
    import torch
    return torch


def _dev(x):
    return _torch().from_numpy(np.ascontiguousarray(x)).cuda()


def _workload(name, iters=16):
    n, U, K, deps, b, T, own = {**CASES, **STREAMED}[name]
    rng = np.random.Generator(np.random.PCG64(2600 + list({**CASES, **STREAMED}).index(name)))
    model = synth.make_model(rng, n, U, K, deps, b if own else 1, 1.0, 1.0, uniform_D=False)
    obs, act = synth.sample_sequences(rng, model, b, T)
    return synth.Workload(name, ["fpi", "vmp", "mmp"], model, obs, act, iters), rng


def _coupled(name, iters=16):
    n, U, K, deps, lists, b, T, own = {**COUPLED, **FILTER_LISTS}[name]
    rng = np.random.Generator(np.random.PCG64(2650 + len(name)))
    model = synth.make_model(rng, n, U, K, deps, b if own else 1, 1.0, 1.0, uniform_D=False, bdeps=lists)
    obs, act = synth.sample_sequences(rng, model, b, T)
    return synth.Workload(name, ["fpi", "vmp", "mmp"], model, obs, act, iters), rng


def _run(pm, kernel, algo, *args, **kw):
    """The call's result, and that `kernel` (by its profile name) ran it."""
    bi.bi_profile_begin()
    q = (pm.infer_soft if kw.pop("soft", False) else pm.infer)(algo, *args, **kw)
    _torch().cuda.synchronize()
    names = set(bi.bi_profile_end()) - {"soft_ll"}
    assert names == {kernel}, names
    return q.cpu().numpy()


def kernel_of(kind, algo, T=2):
    """The profile name of the kernel that a call of CASES ("resident"), COUPLED
    or STREAMED runs."""
    if algo == "fpi":
        return "agent_filter_resident"
    return "agent_window_" + ("resident" if T == 1 else kind)


def _vs_oracle(name, kind, algo, w, rng):
    print(f"[gpu] {name} {algo} b={w.b} T={w.T}", flush=True)
    pm = bi.PackedModel(w.model)
    kernel = kernel_of(kind, algo, w.T)
    try:
        q = _run(pm, kernel, algo, _dev(w.obs), _dev(w.act), w.iters)
        check_invariants(w, q)
        err = float(np.abs(q - oracle.infer(algo, w.model, w.obs, w.act, w.iters)).max())
        # a first-step prior with zeros, and a damped update
        prior = synth.random_prior(rng, w.model.n, w.b, p_zero=0.3)
        qp = _run(pm, kernel, algo, _dev(w.obs), _dev(w.act), 5, prior=_dev(prior), damping=0.6)
        errp = float(np.abs(qp - oracle.infer(algo, w.model, w.obs, w.act, 5, prior=prior, damping=0.6)).max())
        print(f"[gpu]   vs oracle {err:.3e}, prior and damping {errp:.3e}", flush=True)
        assert err <= TOL and errp <= TOL
    finally:
        pm.close()


@pytest.mark.parametrize("algo", ["fpi", "vmp", "mmp"])
@pytest.mark.parametrize("name", list(CASES))
def test_resident_vs_oracle(name, algo):
    _vs_oracle(name, "resident", algo, *_workload(name))


def form_workload(i, iters=6):
    n, U, deps, lists, T, *_ = FORMS[i]
    rng = np.random.Generator(np.random.PCG64(2700 + i))
    model = synth.make_model(rng, n, U, [3] * len(deps), deps, 2, 1.0, 1.0, uniform_D=False, bdeps=lists)
    obs, act = synth.sample_sequences(rng, model, 2, T)
    return synth.Workload(f"form{i}", ["fpi", "vmp", "mmp"], model, obs, act, iters), rng


@pytest.mark.parametrize("algo", ["fpi", "vmp", "mmp"])
@pytest.mark.parametrize("form", range(len(FORMS)))
def test_resident_forms(form, algo):
    w, rng = form_workload(form)
    _vs_oracle(f"{w.name} {FORMS[form]}", "coupled" if FORMS[form][3] else "resident", algo, w, rng)


@pytest.mark.parametrize("algo", ["vmp", "mmp"])
@pytest.mark.parametrize("name", list(STREAMED))
def test_streamed_vs_oracle(name, algo):
    _vs_oracle(name, "streamed", algo, *_workload(name, iters=6))


@pytest.mark.parametrize("name,algo", [(n, a) for n in COUPLED for a in ("fpi", "vmp", "mmp")] + [("long_lists", "fpi")])
def test_resident_coupled(name, algo):
    _vs_oracle(name, "coupled", algo, *_coupled(name))


@pytest.mark.parametrize("name,algo", [(n, a) for n in ("rank3_subsets", "groups") for a in ("fpi", "vmp", "mmp")]
                         + [("rank4_three_columns", "vmp"), ("streamed_steps", "mmp")])
def test_resident_soft(name, algo):
    w, rng = _workload(name)
    print(f"[gpu] {name} soft {algo}", flush=True)
    pm = bi.PackedModel(w.model)
    kernel = kernel_of("streamed" if name in STREAMED else "resident", algo)
    try:
        so = synth.soft_obs(rng, w.obs, w.model.K, confidence=0.5)
        q = _run(pm, kernel, algo, _dev(so), _dev(w.act), w.iters, soft=True)
        ref = oracle.infer_soft(algo, w.model, so.astype(np.float64), w.act, w.iters)
        assert float(np.abs(q - ref).max()) <= TOL
        one = _run(pm, kernel, algo, _dev(synth.one_hot_obs(w.obs, w.model.K)), _dev(w.act), w.iters, soft=True)
        assert np.array_equal(one, _run(pm, kernel, algo, _dev(w.obs), _dev(w.act), w.iters))
    finally:
        pm.close()


@pytest.mark.parametrize("algo", ["fpi", "vmp", "mmp"])
def test_resident_wide_logs(algo):
    """Exact zeros in A (logs of -36.8 beside ordinary ones) over several
    modalities: the softmax spans 1e-60 and its shift is not this sweep's
    maximum."""
    rng = np.random.Generator(np.random.PCG64(2690))
    model = synth.make_model(rng, [6, 5], [2, 2], [4] * 5, [[0, 1]] * 5, 8, 0.5, 0.5, sparsity=0.5, uniform_D=False)
    obs, act = synth.sample_sequences(rng, model, 8, 6)
    print(f"[gpu] wide logs {algo}", flush=True)
    pm = bi.PackedModel(model)
    try:
        q = _run(pm, kernel_of("resident", algo), algo, _dev(obs), _dev(act), 4)
        assert float(np.abs(q - oracle.infer(algo, model, obs, act, 4)).max()) <= TOL
    finally:
        pm.close()


def test_longest_filter_window():
    """The longest window that the agent-resident family takes, and the first
    that it refuses (before any launch): 24 bytes per state and step."""
    rng = np.random.Generator(np.random.PCG64(2691))
    model = synth.make_model(rng, [8, 6], [3, 1], [5, 7, 4], [[0, 1]] * 3, 1, 1.0, 1.0, uniform_D=False)
    obs, act = synth.sample_sequences(rng, model, 1, 500)
    print("[gpu] fpi b=1 T=480, 500", flush=True)
    pm = bi.PackedModel(model)
    try:
        o, u = np.ascontiguousarray(obs[:, :480]), np.ascontiguousarray(act[:, :479])
        q = _run(pm, kernel_of("resident", "fpi"), "fpi", _dev(o), _dev(u), 4)
        assert float(np.abs(q - oracle.infer("fpi", model, o, u, 4)).max()) <= TOL
        with pytest.raises(bi.BiError) as ei:
            pm.infer("fpi", _dev(obs), _dev(act), 4)
        assert ei.value.code == bi.BI_ERR_UNSUPPORTED
    finally:
        pm.close()
