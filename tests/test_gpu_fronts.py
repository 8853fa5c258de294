"""GPU parity of the front search (8 x 16 tables, calls of more than 2^17 (request, GPU) pairs or more
than 4,096 GPUs), at the sizes and inputs where its steps change:
chunks of requests and of hosts, fronts longer than a bucket's steps (built in the pool, or not
at all), requests and tables that are scored against every GPU, groups that share a sort slot,
and the shapes on either side of the rule that sends a call to it.

Flags and indices must match the oracle exactly and energies within 1e-5; a different index is
accepted only as a near-tie judged by the oracle's float64 energies (oracle/check.py); inputs
with exact ties must give the lowest index."""
import numpy as np
import pytest

import oracle
from oracle.check import check_placements
from paper_2606_30391_amd import workloads as W

torch = pytest.importorskip("torch")
pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")]


def parity(inp, label, exact=False, sel=None):
    from paper_2606_30391_amd import festina as F
    R = inp["requests"]["n_requests"]
    print(f"[gpu] fronts: {label}: R={R} G={inp['gpus']['n_gpus']} W={inp['gpus']['n_waves']} "
          f"M={inp['lut']['n_models']}", flush=True)
    dp = F.DevicePlacement(inp, "cuda")
    for t in (dp.choice, dp.feasible, dp.energy):
        t.fill_(7)                                  # an unwritten entry cannot pass
    dp.run()
    torch.cuda.synchronize()
    got = dp.results()
    sel = np.arange(R) if sel is None else sel
    ref = oracle.score_placements(inp, sel)
    rep = check_placements(inp, sel, ref, tuple(x[sel] for x in got))
    print(f"      {rep}", flush=True)
    assert rep.ok, str(rep)
    if exact:
        assert rep.near_ties == 0 and np.array_equal(got[0][sel], ref[0]), label
    return got


def tiny(seed, **kw):
    kw = dict(dict(R=400, G=40, M=2, NS=8, NF=16, W=2), **kw)
    return W.make_tiny_placement(np.random.default_rng(seed), **kw)


def rising_load(inp, rows=32):
    """Decode latencies that fall with the batch row, the same at every level: a loaded GPU is
    never dominated by a lighter one, so every distinct row stays in every cell's front."""
    lut, g = inp["lut"], inp["gpus"]
    r = np.arange(32, dtype=np.float32)[None, :, None, None]
    lut["dc"][:] = 30.0 - 0.5 * r - 0.01 * np.arange(8, dtype=np.float32)[:, None]
    g["batch"][:] = np.arange(g["n_gpus"], dtype=np.int32)[None] % rows
    g["k_dyn_w"][:] = np.linspace(300, 500, g["n_gpus"]).astype(np.float32)
    g["resident"][:] = 0xffffffff
    q = inp["requests"]
    q["slo_tbt_ms"] = np.random.default_rng(1).uniform(12.0, 32.0, q["n_requests"]).astype(np.float32)
    return inp


@pytest.mark.parametrize("R", [1, 15, 16, 17, 127, 128, 129, 1100])
def test_request_chunks(R):
    parity(W.make_placement(2, n_requests=R, n_gpus=4100), f"{R} requests")


@pytest.mark.parametrize("G,caps", [(1, False), (127, True), (128, False), (129, True), (300, True), (1030, False)])
def test_host_chunks(G, caps):
    """Every GPU hosts both models: one, several and partly filled chunks of 128 hosts, and more
    GPUs than one round of the list builder."""
    inp = tiny(11 + G, R=max(400, 2**17 // G + 1), G=G, caps=caps)
    inp["gpus"]["resident"][:] = 3
    parity(inp, f"{G} hosts caps={caps}")


def test_long_fronts_of_few_buckets():
    """Six buckets have room for 64 steps each."""
    parity(rising_load(tiny(21, R=2100, G=64, M=3, W=2, caps=False)), "64 steps per front")


def test_long_fronts_in_the_pool():
    """1,200 buckets have room for 16 steps each: the 30 fronts of one model are built again, longer."""
    inp = tiny(24, R=19000, G=64, M=40, W=30, caps=False)
    other = inp["lut"]["dc"][1:].copy()
    rising_load(inp)
    inp["lut"]["dc"][1:] = other                    # model 0 alone has the falling latencies
    inp["requests"]["model"][::5] = 0
    parity(inp, "30 of 1,200 fronts of 64 steps", sel=np.arange(0, 19000, 11))


def test_more_long_fronts_than_the_pool_holds():
    """1,200 fronts of 64 steps, where the pool has room for 64 of them: which buckets get it depends on
    scheduling, the results do not."""
    inp = rising_load(tiny(22, R=19000, G=64, M=40, W=30, caps=False))
    sel = np.arange(0, 19000, 11)
    got = parity(inp, "1,200 fronts of 64 steps", sel=sel)
    for a, b in zip(got, parity(inp, "the same again", sel=sel)):
        assert np.array_equal(a, b)


def test_fronts_too_long_to_keep():
    """Every cap pair and 32 loads: some cells keep more than 255 candidates."""
    inp = rising_load(tiny(23, R=200, G=2048, M=1, W=1, caps=True))
    parity(inp, "2048 hosts, every cap pair")


@pytest.mark.parametrize("caps", [False, True])
def test_every_gpu_ties(caps):
    """All candidates of a level tie exactly, whatever order the GPUs are pruned in."""
    inp = tiny(31, R=700, G=200, M=2, W=2, caps=caps, ties=True)
    inp["lut"]["p0_w"] = 100.0
    inp["gpus"]["k_dyn_w"][:] = 0.0
    parity(inp, f"ties caps={caps}", exact=True)


def test_equal_keys_at_several_cells_and_gpus():
    """Two frequencies and two SM levels of equal power and latency: the least key is attained at
    several cells; GPUs in descending load order, so the lowest id is not the lightest."""
    inp = tiny(32, R=1500, G=90, M=2, W=2, caps=True)
    lut = inp["lut"]
    lut["freq_level"][:] = np.repeat(lut["freq_level"][::4], 4)
    lut["sm_level"][:] = np.repeat(lut["sm_level"][::2], 2)
    for k in ("pf", "dc"):
        lut[k][:] = np.repeat(np.repeat(lut[k][:, :, ::2, ::4], 2, axis=2), 4, axis=3)
    inp["gpus"]["batch"][:] = -np.sort(-inp["gpus"]["batch"], axis=1)
    inp["gpus"]["k_dyn_w"][:] = 350.0
    parity(inp, "repeated cells", exact=True)


def test_requests_scored_against_every_gpu():
    """No prompt, no output, or a table with negative or tiny latencies, mixed with others."""
    inp = tiny(41, R=3300, M=3, caps=True)
    q = inp["requests"]
    q["pred_out_tokens"][::5] = 0
    q["prompt_tokens"][::7] = 0
    inp["lut"]["pf"][1, 3, 2, 5] = np.float32(1e-30)
    inp["lut"]["dc"][2, 4, 1, 1] = np.float32(-3.0)
    parity(inp, "unusual requests and tables")


@pytest.mark.parametrize("one_slo", [False, True])
@pytest.mark.parametrize("R,kind", [(1, "no prompt"), (20, "no prompt"), (40, "no output"), (70, "no prompt"),
                                    (130, "no prompt"), (130, "no output"), (130, "tiny row"), (130, "negative row")])
def test_requests_without_a_front(R, kind, one_slo):
    """Groups of up to 4, 8 and 16 requests that every hosting GPU is scored for (1,025 of 4,100: several
    rounds of 64, the last one partly filled), with and without one SLO per group, capped GPUs."""
    inp = W.make_placement(2, n_requests=R, n_gpus=4100)
    rng, q, g = np.random.default_rng(R), inp["requests"], inp["gpus"]
    g["cap_pf"], g["cap_dc"] = (rng.integers(0, 8, 4100).astype(np.int8) for _ in range(2))
    q["model"] %= 3
    if kind == "no prompt":
        q["prompt_tokens"][:] = 0
    elif kind == "no output":
        q["pred_out_tokens"][:] = 0
    else:
        inp["lut"]["pf"][:, :, 3, 7] = 1e-30 if kind == "tiny row" else -0.5
    if not one_slo:
        q["slo_ttft_ms"] *= rng.uniform(0.3, 1.5, R).astype(np.float32)
        q["slo_tbt_ms"] *= rng.uniform(0.3, 1.5, R).astype(np.float32)
    parity(inp, f"{kind}, one SLO={one_slo}")


def test_slo_values():
    """TBT SLOs different for every request of a group, and infinite, zero or NaN SLOs."""
    inp = tiny(42, R=3300, M=1, W=1, caps=True)
    q = inp["requests"]
    q["slo_ttft_ms"][::9] = np.inf
    q["slo_tbt_ms"][1::9] = np.inf
    q["slo_tbt_ms"][2::9] = 0.0
    q["slo_tbt_ms"][3::9] = np.nan
    q["slo_ttft_ms"][4::9] = np.nan
    parity(inp, "SLO values")


def test_groups_that_share_a_slot():
    """630 buckets of shuffled requests: more groups in a chunk than sort slots keep apart."""
    parity(tiny(51, R=33000, G=60, M=70, W=9, caps=True), "630 buckets")


@pytest.mark.parametrize("R", [4100, 4104])
def test_either_side_of_the_route(R):
    """2,050 buckets: the front search takes calls of at least 4,104 requests."""
    inp = tiny(52, R=R, G=1400, M=41, W=50, caps=True)
    parity(inp, f"2050 buckets, {R} requests", sel=np.arange(0, R, 6))


def test_a_workspace_without_room_for_fronts():
    """A workspace sized for a call of more waves, which has no fronts, is less than the fronts of
    fewer waves take: the kernels that score every candidate serve the call."""
    from paper_2606_30391_amd import festina as F
    inp = tiny(61, R=13000, G=100, M=32, W=64, caps=True)
    dp = F.DevicePlacement(inp, "cuda")
    more = F.festina_gpus(100, 128, *([None] * 5))
    nbytes = F.festina_placements_workspace_bytes(dp.lut, more, dp.req)
    assert nbytes < dp.ws_bytes
    print(f"[gpu] fronts: workspace of {nbytes} bytes instead of {dp.ws_bytes}", flush=True)
    dp.workspace = torch.empty(nbytes, dtype=torch.uint8, device="cuda")
    dp.ws_bytes = nbytes
    dp.run()
    torch.cuda.synchronize()
    sel = np.arange(0, 13000, 9)
    rep = check_placements(inp, sel, oracle.score_placements(inp, sel), tuple(x[sel] for x in dp.results()))
    assert rep.ok, str(rep)
