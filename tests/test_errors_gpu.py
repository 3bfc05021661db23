"""Failure paths on the GPU: a workspace allocation that fails is reported as
TM_ERR_NO_MEMORY before anything is enqueued, and the library recovers.  The
failure is forced from the host (the TM_TEST_FAIL_ALLOC switch of the
workspace cache); every kernel that does run exits normally."""
import pytest

from gpu_helpers import log, make_input, to_device

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
from paper_2512_04632_amd import _lib as tm  # noqa: E402


def test_failed_allocation_reports_no_memory_and_recovers(monkeypatch):
    log("case: forced workspace allocation failure, 512 x 1536 bf16 AOL t=4")
    X = make_input(512, 1536, 0.8, 2, "bf16")
    ref = to_device(X, "bf16")
    tm.orthogonalize(ref, 4, None, "aol")
    torch.cuda.synchronize()
    tm.release_workspaces()            # every cache empty: the next call must allocate
    x = to_device(X, "bf16")
    keep = x.clone()
    monkeypatch.setenv("TM_TEST_FAIL_ALLOC", "1")
    with pytest.raises(tm.TurboMuonError) as err:
        tm.orthogonalize(x, 4, None, "aol")
    assert err.value.status == tm.TM_ERR_NO_MEMORY
    assert "allocation" in tm.last_error()
    torch.cuda.synchronize()
    assert torch.equal(x, keep)        # nothing was enqueued
    # the allocation-free entry point needs no allocation, so it still runs
    y = x.clone()
    tm.orthogonalize_noalloc(y, 4, None, "aol")
    torch.cuda.synchronize()
    assert torch.equal(y, ref)
    monkeypatch.delenv("TM_TEST_FAIL_ALLOC")
    tm.orthogonalize(x, 4, None, "aol")
    torch.cuda.synchronize()
    assert torch.equal(x, ref)


def test_short_of_memory_takes_a_smaller_workspace(monkeypatch):
    """Refused allocations from the size of the preferred layout on: the call runs on the
    layout with the least padding (same bits), and fp32 also on the fp32 kernels, which need
    less than the padded planes."""
    log("case: workspace allocations refused from a size on")
    g = torch.Generator(device="cuda")
    g.manual_seed(5)
    for dtype, shape, refused, bound in ((torch.bfloat16, (1, 3365, 6105), 185 * 10 ** 6, 0.0),
                                         (torch.float32, (40, 65, 65), 10 * 10 ** 6, 2e-4)):
        # 181 MB on tiles of 64 and 128, 192 MB on 256; 13 MB as planes, 4 MB in fp32
        x = torch.randn(shape, generator=g, device="cuda").to(dtype)
        ref = x.clone()
        tm.orthogonalize(ref, 4, None, "aol")
        torch.cuda.synchronize()
        tm.release_workspaces()
        monkeypatch.setenv("TM_TEST_FAIL_ALLOC", str(refused))
        tm.orthogonalize(x, 4, None, "aol")
        torch.cuda.synchronize()
        monkeypatch.delenv("TM_TEST_FAIL_ALLOC")
        tm.release_workspaces()
        assert float((x.double() - ref.double()).norm() / ref.double().norm()) <= bound
