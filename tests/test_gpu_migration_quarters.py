"""GPU parity of the consolidation search where a wavefront's quarter of the destinations ends:
lanes left over, whole and part batches of records, fewer GPUs than wavefronts, an odd last
source, and budgets whose difference does not fit an int."""
import sys

import numpy as np
import pytest

import oracle
from oracle.check import check_migrations
from paper_2606_30391_amd import workloads as W

torch = pytest.importorskip("torch")
pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")]


def parity(inp, label):
    from paper_2606_30391_amd import festina as F
    G = inp["fleet"]["n_gpus"]
    print(f"[gpu] migration {label}: G={G}", flush=True)
    sys.stdout.flush()
    dm = F.DeviceMigration(inp, "cuda")
    dm.run()
    torch.cuda.synchronize()
    sel = np.unique(np.concatenate([np.arange(min(G, 40)), np.arange(max(0, G - 40), G)]))
    rep = check_migrations(inp, sel, oracle.score_migrations(inp, sel), tuple(x[sel] for x in dm.results()))
    assert not rep.mismatches, rep.mismatches[:5]


@pytest.mark.parametrize("G", [2, 3, 5, 255, 257, 513, 1535, 1537, 1540, 2047, 2049, 3600])
def test_quarter_edges(G):
    parity(W.make_tiny_fleet(np.random.default_rng(7300 + G), G=G, M=3, NS=4, NF=16), "quarters")


@pytest.mark.parametrize("NF", [1, 31, 32])
def test_level_count_limits(NF):
    parity(W.make_tiny_fleet(np.random.default_rng(7400 + NF), G=130, M=3, NS=3, NF=NF), f"{NF} levels")


def test_budgets_beyond_int():
    """Room below every int admits no pair, room above every int admits all."""
    inp = W.make_tiny_fleet(np.random.default_rng(7500), G=70, M=2, NS=3, NF=8, loose=True, huge_budget=True)
    fl = inp["fleet"]
    fl["hbm_mib"][:10] = -2**31
    fl["hbm_cap_mib"] = 2**31 - 1
    fl["sm_permille"][20:30] = 2**31 - 1
    fl["sm_cap_permille"] = 2000
    parity(inp, "budgets")
