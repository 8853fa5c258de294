"""GPU parity of the preferred configurations (App. E) and the fleet's energy waste ratio
(Sec. 3.5.1): the HIP path through the C ABI against the CPU oracle.

Preferred configurations: flags and chosen cells exactly (a different cell only as a
near-tie by the oracle's float64 energies), durations, powers and the two averages within
1e-5 (oracle/check.py).  EWR on the same float32 inputs: per-GPU frequencies exactly,
waste and totals within 1e-9 (both sum in float64).  The chained run (preferred
configurations feeding the EWR) is compared with the oracle's own chain within 1e-5.
"""
import sys

import numpy as np
import pytest

import oracle
from conftest import golden_preferred, load_golden
from oracle.check import check_ewr, check_preferred
from paper_2606_30391_amd import workloads as W

torch = pytest.importorskip("torch")
pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")]


def say(*a):
    print(*a, flush=True)
    sys.stdout.flush()


def device(inp):
    from paper_2606_30391_amd import festina as F
    F.lib()
    return F.DevicePreferred(inp, "cuda")


def parity_preferred(inp, label=""):
    q = inp["llms"]
    say(f"[gpu] preferred {label}: G={q['n_gpus']} K={q['max_inst']} NS={inp['lut']['n_sm']} NF={inp['lut']['n_freq']}")
    dp = device(inp)
    dp.run()
    torch.cuda.synchronize()
    got = dp.results()
    ref = oracle.preferred(inp)
    rep = check_preferred(inp, ref, got)
    say(f"      {rep}")
    assert rep.ok, str(rep)
    return dp, got, ref


def gpu_ewr(n_inst, f_pref, t_ms):
    """EWR on the device from host arrays (a DevicePreferred shell supplies the buffers)."""
    from paper_2606_30391_amd import festina as F
    F.lib()
    G, K = f_pref.shape
    n = torch.from_numpy(np.ascontiguousarray(n_inst, np.int32)).cuda()
    f = torch.from_numpy(np.ascontiguousarray(f_pref, np.float32).reshape(-1)).cuda()
    t = torch.from_numpy(np.ascontiguousarray(t_ms, np.float32).reshape(-1)).cuda()
    fg = torch.empty(G, dtype=torch.float32, device="cuda")
    wg = torch.empty(G, dtype=torch.float64, device="cuda")
    tot = torch.empty(3, dtype=torch.float64, device="cuda")
    out = F.festina_ewr(F._ptr(fg), F._ptr(wg), F._ptr(tot))
    nb = F.festina_ewr_workspace_bytes(G)
    ws = torch.empty(nb, dtype=torch.uint8, device="cuda")
    F.festina_fleet_ewr(G, K, n, f, t, out, ws, nb)
    torch.cuda.synchronize()
    return fg.cpu().numpy(), wg.cpu().numpy(), tot.cpu().numpy()


def test_preferred_fleet_full_size_and_chained_ewr():
    inp = W.make_llms()
    dp, got, ref = parity_preferred(inp, label="2048 GPUs")
    q = inp["llms"]
    live = np.arange(q["max_inst"])[None, :] < q["n_inst"][:, None]
    assert 0.6 < got["feasible"][live].mean() < 1.0
    # the chain: EWR of the device's own preferred frequencies and times
    fg, wg, tot = dp.ewr_results()
    of, ow, (ow_tot, oo_tot, oewr) = oracle.fleet_ewr(q["n_inst"], ref["f_pref"].astype(np.float32),
                                                      (ref["t_p"] + ref["t_d"]).astype(np.float32))
    say(f"      chained EWR {tot[2]:.6f} (oracle chain {oewr:.6f})")
    assert abs(tot[1] - oo_tot) <= 1e-5 * oo_tot
    assert abs(tot[0] - ow_tot) <= 1e-5 * oo_tot
    assert abs(tot[2] - oewr) <= 1e-5


@pytest.mark.parametrize("extra", [100, 200])
def test_preferred_fleet_seeds(extra):
    parity_preferred(W.make_llms(seed=W.LLMS_SEED + extra, n_gpus=512), label=f"seed +{extra}")


@pytest.mark.parametrize("NS,NF", [(1, 1), (3, 5), (4, 8), (8, 16), (16, 16), (2, 33), (5, 50)])
def test_preferred_table_shapes(NS, NF):
    rng = np.random.default_rng(1100 + NS * 100 + NF)
    parity_preferred(W.make_tiny_llms(rng, G=200, K=3, M=3, NS=NS, NF=NF, nan_cells=True), label="shapes")


def test_preferred_zero_output_and_invalid_slots():
    rng = np.random.default_rng(1200)
    inp = W.make_tiny_llms(rng, G=120, K=3, M=2, NS=4, NF=6, zero_out=True)
    q = inp["llms"]
    q["n_inst"][:5] = [3, 4, -1, 0, 3]
    q["model"][0, 1] = 9
    q["batch"][4, 2] = -2
    q["avg_in_tokens"][5, 0] = 0
    q["avg_out_tokens"][6, 0] = -1
    dp, got, ref = parity_preferred(inp, label="zero output, invalid slots")
    assert not got["feasible"][1:4].any() and got["feasible"][0, 1] == 0 and got["feasible"][4, 2] == 0


@pytest.mark.parametrize("variant", [None, "TTFT SLO equal to the fastest prefill",
                                     "TBT SLO equal to the best decode latency"])
def test_preferred_worked_example(variant):
    inp, exp, d = golden_preferred(variant)
    dp = device(inp)
    dp.run_preferred()
    torch.cuda.synchronize()
    got = dp.results()
    for f in ("sm_p", "f_p", "sm_d", "f_d", "feasible"):
        assert got[f][0, 0] == exp[f], f
    for f, key in (("t_p", "t_p_ms"), ("t_d", "t_d_ms"), ("p_p", "p_p_w"), ("p_d", "p_d_w")):
        if f in exp:
            assert got[key][0, 0] == np.float32(exp[f]), f
    for f in ("sm_pref", "f_pref"):
        if f in exp:
            num, den = exp[f]
            assert got[f][0, 0] == pytest.approx(num / den, rel=1e-6), f


def test_ewr_worked_example():
    d = load_golden("preferred_worked_example.json")["ewr"]
    fg, wg, tot = gpu_ewr(np.array(d["n_inst"]), np.array(d["f_pref"]), np.array(d["t_ms"]))
    e = d["expected"]
    assert list(fg) == e["f_gpu"] and list(wg) == e["waste_gpu"]
    assert tot[0] == e["e_waste"] and tot[1] == e["e_optimal"]
    assert tot[2] == pytest.approx(e["ewr"][0] / e["ewr"][1], rel=1e-15)


@pytest.mark.parametrize("G,K", [(1, 1), (7, 3), (255, 4), (256, 4), (257, 2), (70001, 4)])
def test_ewr_random_fleets(G, K):
    rng = np.random.default_rng(1300 + G)
    n = rng.integers(0, K + 1, G).astype(np.int32)
    n[rng.random(G) < 0.01] = K + 2                       # invalid counts: GPU left empty
    f = rng.uniform(0.5, 1.0, (G, K)).astype(np.float32)
    t = rng.uniform(1.0, 3000.0, (G, K)).astype(np.float32)
    f[rng.random((G, K)) < 0.05] = np.nan
    t[rng.random((G, K)) < 0.02] = np.inf
    got = gpu_ewr(n, f, t)
    ref = oracle.fleet_ewr(n, f, t)
    rep = check_ewr(ref, got)
    say(f"[gpu] EWR G={G} K={K}: {rep}")
    assert rep.ok, str(rep)
    again = gpu_ewr(n, f, t)
    assert all(np.array_equal(x, y, equal_nan=True) for x, y in zip(got, again))


def test_ewr_many_slots_per_gpu():
    """More than 8 instance slots per GPU: the slot loop that reads up to the count."""
    rng = np.random.default_rng(1400)
    G, K = 3000, 11
    n = rng.integers(0, K + 1, G).astype(np.int32)
    f = rng.uniform(0.5, 1.0, (G, K)).astype(np.float32)
    t = rng.uniform(1.0, 3000.0, (G, K)).astype(np.float32)
    f[rng.random((G, K)) < 0.05] = np.nan
    rep = check_ewr(oracle.fleet_ewr(n, f, t), gpu_ewr(n, f, t))
    say(f"[gpu] EWR G={G} K={K}: {rep}")
    assert rep.ok, str(rep)


# 16 lanes per slot: 64, 65, 128 and 129 cells are the edges of 4, 8 and 16 cells per lane;
# 1, 15, 16 and 17 slots those of a block
@pytest.mark.parametrize("G,K,NS,NF", [(1, 1, 4, 16), (5, 3, 5, 13), (4, 4, 8, 16), (17, 1, 3, 43)])
def test_preferred_lanes_per_slot(G, K, NS, NF):
    rng = np.random.default_rng(1700 + NS * NF)
    parity_preferred(W.make_tiny_llms(rng, G=G, K=K, M=2, NS=NS, NF=NF, nan_cells=True), label="lanes per slot")


# one block: two GPUs of a thread at once (1,024 apart), four slots per load where they are aligned
@pytest.mark.parametrize("G,K,shift", [(1023, 4, 0), (1025, 4, 1), (2049, 8, 0), (3100, 8, 3), (2500, 5, 0)])
def test_ewr_single_block(G, K, shift):
    from paper_2606_30391_amd import festina as F
    F.lib()
    rng = np.random.default_rng(1800 + G)
    n = rng.integers(0, K + 1, G).astype(np.int32)
    f = rng.uniform(0.5, 1.0, (G, K)).astype(np.float32)
    t = rng.uniform(1.0, 3000.0, (G, K)).astype(np.float32)
    f[rng.random((G, K)) < 0.05] = np.nan
    dev = [torch.empty(G * K + shift, dtype=torch.float32, device="cuda")[shift:] for _ in range(2)]
    for d, h in zip(dev, (f, t)):
        d.copy_(torch.from_numpy(h.reshape(-1)))
    fg = torch.empty(G, dtype=torch.float32, device="cuda")
    wg = torch.empty(G, dtype=torch.float64, device="cuda")
    tot = torch.empty(3, dtype=torch.float64, device="cuda")
    nb = F.festina_ewr_workspace_bytes(G)
    ws = torch.empty(nb, dtype=torch.uint8, device="cuda")
    F.festina_fleet_ewr(G, K, torch.from_numpy(n).cuda(), dev[0], dev[1],
                        F.festina_ewr(F._ptr(fg), F._ptr(wg), F._ptr(tot)), ws, nb)
    torch.cuda.synchronize()
    rep = check_ewr(oracle.fleet_ewr(n, f, t), (fg.cpu().numpy(), wg.cpu().numpy(), tot.cpu().numpy()))
    say(f"[gpu] EWR G={G} K={K} shift={shift}: {rep}")
    assert rep.ok, str(rep)
