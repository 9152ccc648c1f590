"""Workspace of a small ragged batch: shorter work items, which spread it over the chip, take more top-k lists; they
are bounded, whatever k, and a workspace that holds only the lists of the tuning table's item lengths is planned with
those, with the same results."""
import numpy as np
import pytest

from gpu_harness import log

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

N, L, NQ = 2_000_000, 64, 512
MB = 1 << 20


@pytest.fixture(scope="module")
def world():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1707_00516_amd import fid_row_words
    from paper_1707_00516_amd.torch_api import Context
    ctx = Context(0)
    g = torch.Generator(device="cuda").manual_seed(N)
    rows = torch.randint(-2**63, 2**63 - 1, (N + NQ, fid_row_words(L)), generator=g, device="cuda", dtype=torch.int64)
    rows[:, 1:] = 0
    yield ctx, ctx.build_db(rows[:N].contiguous(), L), rows[N:].contiguous()
    ctx.sync()
    ctx.close()


def _lists_bytes(tiles, k):
    """Lists and fill counts of one job of NQ queries against N references in items of `tiles` 512-reference tiles."""
    owners = 8 * -(-(-(-N // 512)) // tiles)
    return NQ * owners * (8 * k + 4)


@pytest.mark.parametrize("k", [1, 32, 128])
def test_lists_are_bounded(world, k):
    from paper_1707_00516_amd import FidJob, fid_batch_workspace_bytes
    ctx, db, q = world
    out = torch.empty((NQ, k), dtype=torch.int64, device="cuda")
    jobs = [FidJob(db.handle, 0, N, q.data_ptr(), NQ, 0, out.data_ptr(), out.data_ptr())]
    need = fid_batch_workspace_bytes(ctx.handle, jobs, k)
    # beside the lists: seed counts, staged queries, tables
    rest = NQ * 16384 * 4 + 4 * MB
    log(f"k={k}: {need / MB:.0f} MB, of which lists at most {max(256 * MB, _lists_bytes(128, k)) / MB:.0f}")
    assert need <= max(256 * MB + 12 * MB, _lists_bytes(128, k)) + rest


def test_smaller_workspace_takes_the_tables_lengths(world, k=32):
    from paper_1707_00516_amd import (FID_ENOMEM, FidError, FidJob, fid_batch_create, fid_batch_destroy, fid_batch_run,
                                      fid_batch_workspace_bytes)
    ctx, db, q = world
    got = []
    for share in (1, 2, 16):
        cnt = torch.empty((NQ, k), dtype=torch.int32, device="cuda")
        idx = torch.empty((NQ, k), dtype=torch.int64, device="cuda")
        jobs = [FidJob(db.handle, 0, N, q.data_ptr(), NQ, 0, cnt.data_ptr(), idx.data_ptr())]
        ws = torch.empty(fid_batch_workspace_bytes(ctx.handle, jobs, k) // share, dtype=torch.uint8, device="cuda")
        if share == 16:  # not even the seed counts fit
            with pytest.raises(FidError) as e:
                fid_batch_create(ctx.handle, jobs, k, None, ws.data_ptr(), ws.numel())
            assert e.value.status == FID_ENOMEM
            break
        b = fid_batch_create(ctx.handle, jobs, k, None, ws.data_ptr(), ws.numel())
        fid_batch_run(b, False)
        ctx.sync()
        fid_batch_destroy(b)
        got.append((cnt, idx))
    want = ctx.compare_topk(db, q, 0, k)
    ctx.sync()
    for cnt, idx in got:
        assert torch.equal(cnt, want[0]) and torch.equal(idx, want[1])
    assert np.all(got[0][0].cpu().numpy()[:, 0] >= 0)
