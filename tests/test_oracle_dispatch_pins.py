"""Pins of the current-frequency dispatch oracle (Sec. 3.3, Phases One to Three).

* a hand-worked example and five variants (2% margin in and out, equal memory, the F_max
  fallback by earliest availability, a new GPU, nothing feasible),
* enumeration on tiny random instances (tests/brute.py: list every operating point, the
  2% tie set, the stability order as a sort key, the fallback as the minimum of a list),
* the stability tie-break against numpy.lexsort on exact ties, scaling of power,
* invariants on the dispatch workload.
"""
import numpy as np
import pytest

import oracle
from brute import brute_dispatch, dispatch_points, point_energy
from conftest import golden_dispatch, load_golden
from paper_2606_30391_amd import workloads as W

VARIANTS = [v["name"] for v in load_golden("dispatch_worked_example.json")["variants"]]


def _expect(got, exp):
    g, k, j, ph, e = got
    assert (int(g[0]), int(k[0]), int(j[0]), int(ph[0])) == (exp["gpu"], exp["freq_level"], exp["sm_level"],
                                                              exp["phase"])
    assert (e[0] == np.inf) if exp["energy_mj"] is None else (e[0] == exp["energy_mj"])


@pytest.mark.parametrize("variant", [None] + VARIANTS)
def test_dispatch_worked_example(variant):
    inp, exp, d = golden_dispatch(variant)
    _expect(oracle.dispatch(inp), exp)
    _expect(brute_dispatch(inp), exp)


@pytest.mark.parametrize("seed", range(6))
def test_dispatch_matches_enumeration(seed):
    rng = np.random.default_rng(9000 + seed)
    for case in range(40):
        inp = W.make_tiny_dispatch(rng, ties=(case % 4 == 0))
        o, b = oracle.dispatch(inp), brute_dispatch(inp)
        for x, y, name in zip(o[:4], b[:4], ("gpu", "freq", "sm", "phase")):
            assert np.array_equal(x, y), (seed, case, name)
        assert np.array_equal(o[4], b[4]), (seed, case)


def test_stability_tie_break_is_a_lexicographic_order():
    """Exactly equal energies everywhere (one table value, no dynamic power): the choice is
    the lexsort maximum of (free memory, free SMs, -id) over the feasible GPUs."""
    rng = np.random.default_rng(91)
    checked = 0
    for it in range(100):
        inp = W.make_tiny_dispatch(rng, R=4, G=8, M=1, NS=3, NF=3, S=2, ties=True)
        inp["avail"]["k_dyn_w"][:] = 0.0
        if it % 2:                        # equal free memory everywhere: the free SMs decide
            inp["avail"]["mem_free_mib"][:] = inp["avail"]["mem_free_mib"][:1]
        g, k, j, ph, e = oracle.dispatch(inp)
        for r in range(4):
            pts = [(gg, ta, sm, mem, b) for gg, ta, sm, mem, b in dispatch_points(inp, r)
                   if point_energy(inp, r, sm, int(inp["avail"]["freq_cur"][gg]), ta, b, 0.0) is not None]
            if not pts:
                assert ph[r] != 1
                continue
            ids = np.array([p[0] for p in pts])
            order = np.lexsort((ids, -np.array([p[2] for p in pts]), -np.array([p[3] for p in pts])))
            assert ph[r] == 1 and g[r] == ids[order[0]]
            checked += 1
    assert checked > 100


def test_dispatch_power_scaling():
    rng = np.random.default_rng(92)
    inp = W.make_tiny_dispatch(rng, R=200, G=10, M=2, NS=4, NF=5, S=3)
    a = oracle.dispatch(inp)
    inp["lut"]["p0_w"] *= 2.0
    inp["avail"]["k_dyn_w"] = (inp["avail"]["k_dyn_w"] * 2).astype(np.float32)
    inp["avail"]["k_new_w"] *= 2.0
    b = oracle.dispatch(inp)
    for x, y in zip(a[:4], b[:4]):
        assert np.array_equal(x, y)
    assert np.array_equal(a[4] * 2, b[4])


def test_dispatch_workload_invariants():
    inp = W.make_dispatch(n_requests=600, n_gpus=96)
    g, k, j, ph, e = oracle.dispatch(inp)
    counts = np.bincount(ph, minlength=4)
    assert counts[1] > 300 and counts.min() >= 0
    b = brute_dispatch(inp)
    for x, y in zip((g, k, j, ph), b[:4]):
        assert np.array_equal(x, y)
    assert np.array_equal(e, b[4])


def test_dispatch_negative_energies():
    """Negative power terms: the 2% band is taken on |E_min|, so the least-energy GPU is
    always inside it and the stability order still decides among its neighbours."""
    rng = np.random.default_rng(93)
    for _ in range(30):
        inp = W.make_tiny_dispatch(rng, R=30, G=8, M=2, NS=3, NF=4, S=2)
        inp["lut"]["p0_w"] = float(np.float32(rng.uniform(0.0, 5.0)))
        inp["avail"]["k_dyn_w"] = (-rng.uniform(0.0, 500.0, 8)).astype(np.float32)
        o, b = oracle.dispatch(inp), brute_dispatch(inp)
        for x, y in zip(o, b):
            assert np.array_equal(x, y)
        assert np.any(o[4][o[3] == 1] < 0)


@pytest.mark.parametrize("where", ["k_dyn_w", "table"])
def test_dispatch_energy_of_minus_infinity(where):
    """A GPU whose energy is -inf (a -inf power coefficient or decode latency): no energy lies within
    2% of E_min (the bound E_min + 0.02 |E_min| is NaN), so a request that this GPU can serve is
    placed nowhere (phase 0); a request of another model is not touched."""
    lut = {"n_models": 2, "n_rows": 32, "n_sm": 1, "n_freq": 1, "sm_level": W.sm_levels(1),
           "freq_level": W.freq_levels(1), "pf": np.full((2, 32, 1, 1), 4.0, np.float32),
           "dc": np.full((2, 32, 1, 1), 2.0, np.float32), "p0_w": 50.0}
    avail = {"n_gpus": 3, "n_steps": 1, "freq_cur": np.zeros(3, np.int32), "batch": np.array([1, 2, 3], np.int32),
             "k_dyn_w": np.full(3, 200.0, np.float32), "resident": np.array([[1], [3], [2]], np.uint32),
             "t_avail_ms": np.zeros((3, 1), np.float32), "mem_free_mib": np.full((3, 1), 100, np.int32),
             "sm_free": np.zeros((3, 1), np.int32), "kv_kib_per_token": np.ones(2, np.int32), "k_new_w": 100.0}
    if where == "k_dyn_w":
        avail["k_dyn_w"][0] = -np.inf
    else:
        lut["dc"][0, 1] = -np.inf                       # the batch row of GPU 0
    requests = {"n_requests": 2, "model": np.array([0, 1], np.int32), "wave": None,
                "prompt_tokens": np.full(2, 8, np.int32), "pred_out_tokens": np.full(2, 10, np.int32),
                "slo_ttft_ms": np.full(2, 1e3, np.float32), "slo_tbt_ms": np.full(2, 1e3, np.float32)}
    inp = {"lut": lut, "avail": avail, "requests": requests}
    g, k, j, ph, e = oracle.dispatch(inp)
    assert (g[0], k[0], j[0], ph[0], e[0]) == (-1, -1, -1, 0, np.inf)
    assert ph[1] == 1 and g[1] == 1 and np.isfinite(e[1])
    (wg, _, _, wph, _), st = oracle.dispatch_waves(inp, [0, 2])
    assert wg.tolist() == [-1, 1] and wph.tolist() == [0, 1]
    assert st["batch"].tolist() == [1, 3, 3]
