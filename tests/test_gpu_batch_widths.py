"""A batch whose members have different window half-widths (GPU).

Members of half-width 4 and of others share the launches of the mesh passes;
each member's trajectory is bitwise the one it has alone, for batches of all, of
some and of none of half-width 4.
"""
import pytest

from test_gpu_batch import _alone, _member, _replicas, _same

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("widths", [(4, 4, 4), (4, 3, 5), (3, 6, 3)])
def test_half_widths_in_one_batch(widths, precision):
    import torch

    from paper_1303_4523_amd.batch import Batch
    reps = _replicas([0, 1, 2], n_max=5000)
    for s, p in zip(reps, widths):
        s.meta["enuf"] = dict(s.meta["enuf"], p=p)
    alone = [_alone(s, 3, precision, parts=1) for s in reps]
    b = Batch(precision)
    mem = [_member(s, precision, parts=1) for s in reps]
    for m in mem:
        b.add(*m, first_step=1)
    b.run(3)
    torch.cuda.synchronize()
    for m, ref in zip(mem, alone):
        assert m[0].status() == 0
        assert _same([x.cpu().numpy() for x in m[1:]] + [m[0].energy().cpu().numpy()], ref)
    b.close()
