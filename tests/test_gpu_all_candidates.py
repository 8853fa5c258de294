"""GPU parity of the placement kernels that score every candidate, on the shapes that stay with them:
8 x 16 tables with few requests per (wave, model) on more than 4,096 GPUs (one, two or four
wavefronts per tile by the number of requests), and other tables with too many (request, GPU)
pairs for the one-launch kernel; with the bucket counts scanned inside the scatter or by their
own kernel (more than 8,192 buckets)."""
import numpy as np
import pytest

import oracle
from oracle.check import check_placements
from paper_2606_30391_amd import workloads as W

torch = pytest.importorskip("torch")
pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")]


def sampled_parity(inp, label, n=250):
    from paper_2606_30391_amd import festina as F
    R = inp["requests"]["n_requests"]
    print(f"[gpu] all candidates {label}: R={R} G={inp['gpus']['n_gpus']}", flush=True)
    dp = F.DevicePlacement(inp, "cuda")
    dp.run()
    torch.cuda.synchronize()
    got = dp.results()
    sel = np.sort(np.random.default_rng(R).choice(R, min(n, R), replace=False))
    rep = check_placements(inp, sel, oracle.score_placements(inp, sel), tuple(x[sel] for x in got))
    print(f"      {rep}", flush=True)
    assert rep.ok, str(rep)
    assert np.all((got[1] == 1) == (got[0] >= 0)) and np.all(np.isinf(got[2][got[1] == 0]))


@pytest.mark.parametrize("R,M,Wn", [(6007, 70, 40), (6007, 70, 60), (20011, 70, 100), (40009, 70, 160)])
@pytest.mark.parametrize("one_slo", [False, True])
def test_eight_by_sixteen_sparse_buckets_on_a_large_fleet(R, M, Wn, one_slo):
    rng = np.random.default_rng(R + Wn)
    inp = W.make_tiny_placement(rng, R=R, G=4100, M=M, NS=8, NF=16, W=Wn, caps=True)
    assert M * Wn > 1024 + R // 4
    if one_slo:                                     # tiles take the 8x16 kernel's own scoring
        q = inp["requests"]
        q["slo_ttft_ms"] = rng.uniform(20.0, 70.0, M).astype(np.float32)[q["model"]]
        q["slo_tbt_ms"] = rng.uniform(10.0, 45.0, M).astype(np.float32)[q["model"]]
        q["pred_out_tokens"] = rng.integers(1, 300, R).astype(np.int32)
    sampled_parity(inp, f"{M * Wn} buckets")


@pytest.mark.parametrize("M,Wn,NS,NF,G", [(3, 2, 4, 8, 60), (130, 70, 4, 6, 1000), (3, 2, 8, 12, 60), (3, 2, 16, 16, 60)])
@pytest.mark.parametrize("caps", [False, True])
def test_other_tables(M, Wn, NS, NF, G, caps):
    rng = np.random.default_rng(NS + NF + M)
    sampled_parity(W.make_tiny_placement(rng, R=9001, G=G, M=M, NS=NS, NF=NF, W=Wn, caps=caps), f"{NS}x{NF}", n=1500)
