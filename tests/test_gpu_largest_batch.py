"""The largest int32 batch on the GPU: b = min(B + 1, 32) is formed without overflow (it is a table
row, hence an address), so the results are those of a batch of 31, by every kernel that reads one."""
import numpy as np
import pytest

import largest_batch as LB
from paper_2606_30391_amd import workloads as W

torch = pytest.importorskip("torch")
pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")]


def same(run, label):
    print(f"[gpu] largest batch: {label}", flush=True)
    for a, b in zip(run(31), run(LB.INT32_MAX)):
        assert np.array_equal(a, b, equal_nan=a.dtype.kind == "f"), label


def results(dev):
    torch.cuda.synchronize()
    return dev.results()


@pytest.mark.parametrize("shape", [dict(R=60, G=40), dict(R=60, G=40, NS=4, NF=8), dict(R=9001, G=60, NS=4, NF=8),
                                   dict(R=4000, G=60), dict(R=6007, G=4100, M=70, Wn=40)])
def test_placement(shape):
    """The one-launch kernel, the front search and the kernels that score every candidate."""
    from paper_2606_30391_amd import festina as F

    def run(batch):
        d = F.DevicePlacement(LB.placement(batch, **shape), "cuda")
        d.run()
        return results(d)

    same(run, str(shape))


def test_migration_preferred_and_transfer():
    from paper_2606_30391_amd import festina as F

    def migrate(batch):
        d = F.DeviceMigration(LB.fleet(batch), "cuda")
        d.run()
        return results(d)

    def preferred(batch):
        d = F.DevicePreferred(LB.llms(batch), "cuda")
        d.run_preferred()
        torch.cuda.synchronize()
        return [v.cpu().numpy() for v in d.o.values()]

    def moves(batch):
        d = F.DeviceTransfer(LB.transfer(batch), "cuda")
        d.run_costs()
        d.run_moves()
        return results(d)

    same(migrate, "migration")
    same(preferred, "preferred configurations")
    same(moves, "request moves")


@pytest.mark.parametrize("S", [3, 6, 9])
def test_dispatch(S):
    """One snapshot (packed and gathered profiles) and one wave (packed and unpacked kernels)."""
    from paper_2606_30391_amd import festina as F

    def one(batch):
        d = F.DeviceDispatch(LB.dispatch(batch, S), "cuda")
        d.run()
        return results(d)

    def wave(batch):
        inp = LB.dispatch(batch, S)
        d = F.DeviceDispatch(inp, "cuda")
        d.run_waves(np.array([0, inp["requests"]["n_requests"]], np.int32))
        return results(d)

    same(one, f"dispatch, {S} steps")
    same(wave, f"one wave, {S} steps")
