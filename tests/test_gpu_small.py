"""GPU parity of the one-launch placement kernel for small calls (at most 2^17 (request, GPU) pairs
and 4,096 GPUs): at the numbers of GPUs and requests where its wavefronts per request change, for
all table shapes, and against the other searches on the same requests."""
import numpy as np
import pytest

import oracle
from oracle.check import check_placements
from paper_2606_30391_amd import workloads as W

torch = pytest.importorskip("torch")
pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")]


def run(inp):
    from paper_2606_30391_amd import festina as F
    dp = F.DevicePlacement(inp, "cuda")
    for t in (dp.choice, dp.feasible, dp.energy):
        t.fill_(7)                                  # an unwritten entry cannot pass
    dp.run()
    torch.cuda.synchronize()
    return dp.results()


def parity(inp, label):
    R = inp["requests"]["n_requests"]
    print(f"[gpu] small placement {label}: R={R} G={inp['gpus']['n_gpus']}", flush=True)
    got = run(inp)
    rep = check_placements(inp, np.arange(R), oracle.score_placements(inp), got)
    print(f"      {rep}", flush=True)
    assert rep.ok, str(rep)


@pytest.mark.parametrize("R,G", [(1, 1), (3, 63), (5, 64), (7, 65), (2048, 63), (2048, 64), (255, 513), (256, 512),
                                 (257, 510), (2, 1025), (31, 4096), (32, 4096), (16, 4097)])
@pytest.mark.parametrize("caps", [False, True])
def test_gpus_and_requests(R, G, caps):
    rng = np.random.default_rng(R + G)
    parity(W.make_tiny_placement(rng, R=R, G=G, M=2, NS=8, NF=16, W=2, caps=caps), f"caps={caps}")


@pytest.mark.parametrize("NS,NF", [(1, 1), (4, 8), (5, 13), (8, 16), (3, 43), (16, 16)])
@pytest.mark.parametrize("G", [20, 200])
def test_table_shapes(NS, NF, G):
    rng = np.random.default_rng(NS * 50 + NF + G)
    parity(W.make_tiny_placement(rng, R=301, G=G, M=3, NS=NS, NF=NF, W=2, caps=True, nan_cells=True), f"{NS}x{NF}")


@pytest.mark.parametrize("M", [4, 5, 70])
def test_models(M):
    rng = np.random.default_rng(70 + M)
    parity(W.make_tiny_placement(rng, R=200, G=90, M=M, NS=8, NF=16, W=3, caps=True), f"{M} models")


def same_in_a_small_call(big, n=150):
    """Whatever serves the larger call, its first n requests have the same results in a call of
    their own, bit for bit."""
    want = run(big)
    q = big["requests"]
    for k, v in q.items():
        if isinstance(v, np.ndarray):
            q[k] = np.ascontiguousarray(v[:n])
    q["n_requests"] = n
    for name, a, b in zip(("choice", "feasible", "energy"), want, run(big)):
        assert np.array_equal(a[:n], b), name


@pytest.mark.parametrize("cfg,G", [(2, 64), (3, 200), (4, 333)])
def test_same_results_as_the_larger_call(cfg, G):
    """A request's result does not depend on the size of the call it came with."""
    same_in_a_small_call(W.make_placement(cfg, n_requests=40000, n_gpus=G))


@pytest.mark.parametrize("entry", ["tiny prefill", "negative prefill", "negative decode", "no prompt, no output",
                                   "long fronts"])
def test_same_results_where_requests_have_no_front(entry):
    """Nor on whether its (wave, model) has a front: unusual table entries and requests, and more
    long fronts than there is room for, which the larger call serves in other ways."""
    big = W.make_placement(4 if entry == "long fronts" else 3, n_requests=20000, n_gpus=200)
    lut, q = big["lut"], big["requests"]
    if entry == "tiny prefill":
        lut["pf"][::2, 31, 7, 15] = 1e-30
        lut["pf"][1::2, 3, 2, 5] = 1e-30
    elif entry == "negative prefill":
        lut["pf"][::2, 31, 7, 15] = -1.0
        lut["pf"][1::2, 3, 2, 5] = -1.0
    elif entry == "negative decode":
        lut["dc"][::2, 3, 2, 5] = -1.0
        lut["dc"][1::2, 31, 7, 15] = -1.0
    elif entry == "no prompt, no output":
        q["prompt_tokens"][::3] = 0
        q["pred_out_tokens"][::4] = 0
    else:                                           # 2,048 fronts of 32 steps or more
        big["gpus"]["resident"][:] = 0xffffffff
        lut["dc"][:] = 30.0 - 0.5 * np.arange(32, dtype=np.float32)[None, :, None, None]
        big["gpus"]["batch"][:] = np.arange(200, dtype=np.int32) % 32
        q["slo_tbt_ms"][:] = 32.0
    same_in_a_small_call(big)


@pytest.mark.parametrize("caps", [False, True])
@pytest.mark.parametrize("p0", [0.0, 100.0])
def test_same_results_with_negative_latencies(caps, p0):
    """Negative decode entries turn the order of their rows' Y between hosts, and may make Y and keys
    negative; negative and tiny prefill entries in some rows only.  One -inf entry, and GPUs of negative power.  Bit for bit the
    one-launch kernel's results, which drops no candidate (energies near zero cancel, so they have
    no bound relative to float64)."""
    inp = W.make_placement(4 if caps else 3, seed=77, n_requests=20000, n_gpus=150)
    lut, rng = inp["lut"], np.random.default_rng(43)
    lut["p0_w"] = p0
    lut["dc"][::2, 2:9:3] -= np.float32(60.0)
    lut["dc"][1, 4, 3, 7] = -np.inf
    lut["dc"][1::4][rng.random(lut["dc"][1::4].shape) < 0.01] = np.float32(-3.0)
    lut["pf"][::3, ::5, 4, 9] = np.float32(-2.0)
    lut["pf"][1::3, ::7, 2, 3] = np.float32(1e-30)
    inp["gpus"]["k_dyn_w"][::9] = 0.0
    inp["gpus"]["k_dyn_w"][5::11] = -40.0
    same_in_a_small_call(inp, 5000)
