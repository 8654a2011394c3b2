"""The volume rule in the workspace that its form with device atomics takes: 24 bytes per node
and 4 per edge of a chunk (each array rounded up to 256 bytes), less than the query asks for
large chunks.  Same results, nothing written past it; with less the call is refused."""
import ctypes as C

import numpy as np
import pytest
import torch

import oracle

L = pytest.importorskip("paper_2108_00529_amd._lib", reason="libbgv.so not built")


def least(n, chunk):
    return sum(-(-b // 256) * 256 for b in (8 * n, 16 * n, 4 * chunk))


def test_less_is_refused():
    n, m = 3000, 50_000
    p = L.CdParams(8, 2, 2, 0, m, 0, 1)
    assert L.bgv_community_workspace(n, m, C.byref(p)) > least(n, m)
    some = C.c_void_p(1 << 20)  # not read: the call is refused first
    st = L.bgv_community(n, m, some, C.byref(p), some, some, None, some, least(n, m) - 1, None)
    assert L.bgv_status_string(st) == b"BGV_E_WORKSPACE"


@pytest.mark.gpu
@pytest.mark.parametrize("chunk", [2048, 20_001, 50_000])
def test_small_workspace(chunk):
    n, m = 3000, 50_000
    rng = np.random.default_rng(chunk)
    e = rng.integers(0, n, (m, 2)).astype(np.int32)
    lab, cnt = oracle.bs_community(n, e, 8, 2, 2, chunk, rule=1)
    deg, vol = oracle.degree_volume(lab, cnt, 2)
    p = L.CdParams(8, 2, 2, 0, chunk, 0, 1)
    size, dev = least(n, chunk), torch.device("cuda")
    assert size <= L.bgv_community_workspace(n, m, C.byref(p))
    ws = torch.full((size + 4096,), 0x5a, dtype=torch.uint8, device=dev)
    edges = torch.from_numpy(e).to(dev)
    labels, degree = (torch.empty(n, dtype=torch.int32, device=dev) for _ in range(2))
    volume = torch.empty(n, dtype=torch.int64, device=dev)
    ptr = lambda t: C.c_void_p(t.data_ptr())
    st = L.bgv_community(n, m, ptr(edges), C.byref(p), ptr(labels), ptr(degree), ptr(volume), ptr(ws), size,
                         torch.cuda.current_stream().cuda_stream)
    L.check(st, "bgv_community")
    assert np.array_equal(labels.cpu().numpy(), lab)
    assert np.array_equal(degree.cpu().numpy(), deg)
    assert np.array_equal(volume.cpu().numpy(), vol)
    assert (ws[size:] == 0x5a).all()
