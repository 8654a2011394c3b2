"""A sort of one key has nothing to do: the drawing attributes of one supernode take less time
than those of two, whose keys go through the sort's launches."""
import pytest
import torch

pytestmark = pytest.mark.gpu


def test_one_supernode():
    import paper_2108_00529_amd as bgv
    ms = {}
    for K in (1, 2):
        size = torch.full((K,), 9, dtype=torch.int32, device="cuda")
        group, radius = bgv.draw_supernodes(size)
        assert radius.tolist() == [3.0] * K
        assert group.tolist() == ([10] if K == 1 else [0, 10])
        times = []
        for _ in range(50):
            a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
            torch.cuda.synchronize()
            a.record()
            bgv.draw_supernodes(size)
            b.record()
            torch.cuda.synchronize()
            times.append(a.elapsed_time(b))
        ms[K] = min(times)
    assert ms[1] <= 0.85 * ms[2], ms
