"""Workspaces kept for calls of several sizes: one query fewer than the workspace was sized for, just below the
number of queries from which the other kernel family is faster, is not refused because the faster family's lists are
larger, and gives the result of a call with its own workspace; nor are the queries of a chunked server whose chunks
run another family than its whole database.  A workspace too small for either family's lists is still refused."""
import numpy as np
import pytest

import oracle
from gpu_harness import db_from_bytes, log, pack_rows

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1707_00516_amd.torch_api import Context
    c = Context(0)
    yield c
    c.sync()
    c.close()


def _random_rows(n, L, seed):
    from paper_1707_00516_amd import fid_row_words
    rw = fid_row_words(L)
    g = torch.Generator(device="cuda").manual_seed(seed)
    bits = torch.randint(-2**63, 2**63 - 1, (n, rw), generator=g, device="cuda", dtype=torch.int64)
    live = np.zeros(rw * 64, np.uint8)
    live[:L] = 1
    return bits & torch.from_numpy(np.packbits(live, bitorder="little").view(np.int64)).cuda()


@pytest.mark.parametrize("n,L,n_q", [(540_000, 300, 47), (540_000, 1024, 23), (540_000, 2048, 11), (540_000, 8192, 3)])
def test_one_query_fewer_than_the_workspace_was_sized_for(ctx, n, L, n_q, k=32):
    from paper_1707_00516_amd import FID_ENOMEM, FidError
    log(f"workspace n={n} L={L} n_q={n_q}")
    rows = _random_rows(n + n_q, L, n + L)
    db, q = ctx.build_db(rows[:n].contiguous(), L), rows[n:].contiguous()
    kept = ctx.topk_workspace(db, n_q + 1, k)
    for mode in (oracle.MIXTURE, oracle.IDENTITY):
        want = ctx.compare_topk(db, q, mode, k, ws=ctx.topk_workspace(db, n_q, k))
        got = ctx.compare_topk(db, q, mode, k, ws=kept)
        ctx.sync()
        assert torch.equal(want[0], got[0]) and torch.equal(want[1], got[1]), mode
    # k-slot lists of one owner per query are less than any route needs
    with pytest.raises(FidError) as e:
        ctx.compare_topk(db, q, oracle.MIXTURE, k, ws=kept[:n_q * k * 8])
    assert e.value.status == FID_ENOMEM
    db.close()


def test_noalloc_takes_the_family_that_fits(ctx, n=62_500, L=8, n_q=1025, k=32):
    """Popcount would be faster, but only the fp4 scan's lists fit the fixed scratch array."""
    from paper_1707_00516_amd import fid_compare_topk_noalloc
    log(f"noalloc n={n} L={L} n_q={n_q}")
    rng = np.random.default_rng(n)
    refs = (rng.random((n, L)) < 0.4).astype(np.uint8)
    Q = (rng.random((n_q, L)) < 0.4).astype(np.uint8)
    db, q = db_from_bytes(ctx, refs), pack_rows(ctx, Q)
    cnt = torch.empty((n_q, k), dtype=torch.int32, device="cuda")
    idx = torch.empty((n_q, k), dtype=torch.int64, device="cuda")
    fid_compare_topk_noalloc(ctx.handle, db.handle, q.data_ptr(), n_q, oracle.MIXTURE, k, cnt.data_ptr(),
                             idx.data_ptr())
    ctx.sync()
    wc, wi = oracle.topk(oracle.counts(refs, Q, oracle.MIXTURE), k)
    assert np.array_equal(cnt.cpu().numpy(), wc) and np.array_equal(idx.cpu().numpy(), wi)
    db.close()


def test_server_chunks_of_short_rows(ctx, n=70_000, L=16, n_q=1000, k=4):
    """The server's workspace is sized by whole-database scans (fp4); a chunk of at most 65,536 short rows would run
    popcount, whose lists are larger."""
    from paper_1707_00516_amd.torch_api import Server
    log(f"server n={n} L={L} n_q={n_q}")
    rng = np.random.default_rng(L)
    refs = (rng.random((n, L)) < 0.4).astype(np.uint8)
    Q = (rng.random((n_q, L)) < 0.4).astype(np.uint8)
    db = db_from_bytes(ctx, refs)
    srv = Server(ctx, db, 1 << 30, n_q, k, 2, 0, 1)
    cnt, idx = srv.wait(srv.submit(pack_rows(ctx, Q), oracle.MIXTURE), timeout_us=60_000_000)[:2]
    wc, wi = oracle.topk(oracle.counts(refs, Q, oracle.MIXTURE), k)
    assert np.array_equal(cnt, wc) and np.array_equal(idx, wi)
    srv.close()
    db.close()
