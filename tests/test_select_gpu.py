"""The per-query selections of the top-k (seed bound, direct selection, list
merge) where they change course, against the oracle, bit-exact: fewer
references than k, more equal counts at the k-th place than the selection
holds, up to and beyond one key per thread, narrow and wide workgroups, rows
longer than the histogram has bins, and a row of counts that starts off a
16-byte boundary."""
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


@pytest.mark.parametrize("n_refs,L,n_q,k,kinds", [
    (5, 40, 3, 32, 5), (300, 40, 3, 1024, 300), (5001, 40, 3, 32, 1), (5003, 40, 600, 32, 2),
    (9001, 300, 600, 300, 9001), (16383, 9000, 3, 1024, 16383), (17003, 40, 3, 257, 3), (40001, 64, 530, 7, 40),
    (40003, 5000, 20, 256, 40003), (70001, 64, 1, 1024, 70001)])
def test_selection_edges(ctx, n_refs, L, n_q, k, kinds):
    log(f"selection n_refs={n_refs} L={L} n_q={n_q} k={k} kinds={kinds}")
    rng = np.random.default_rng(n_refs + L)
    few = (rng.random((kinds, L)) < 0.3).astype(np.uint8)  # `kinds` distinct references, repeated
    refs = few[rng.integers(0, kinds, n_refs)] if kinds < n_refs else few
    Q = (rng.random((n_q, L)) < 0.5).astype(np.uint8)
    db, q = db_from_bytes(ctx, refs), pack_rows(ctx, Q)
    for m in (oracle.MIXTURE, oracle.IDENTITY):
        cnt, idx = ctx.compare_topk(db, q, m, k)
        wc, wi = oracle.topk(oracle.counts(refs, Q, m), k)
        assert np.array_equal(cnt.cpu().numpy(), wc) and np.array_equal(idx.cpu().numpy(), wi)
    db.close()


@pytest.mark.parametrize("n_refs,n_q,hits", [(100, 3, 0), (1, 1, 1), (4096, 1, 4096), (4097, 1, 4097), (64, 65, 4160),
                                             (1, 8192, 8192), (1, 8193, 0), (3, 8300, 24900), (50, 64, 3200)])
def test_threshold_hits_csr_edges(ctx, n_refs, n_q, hits):
    """Hits put in order by one launch (at most 4096 of at most 8192 queries)
    and by the sort; every reference of every query is a hit, or none."""
    log(f"hits n_refs={n_refs} n_q={n_q} hits={hits}")
    from paper_1707_00516_amd.torch_api import FidError
    rng = np.random.default_rng(hits)
    L = 90
    refs = np.ones((n_refs, L), np.uint8)
    Q = (rng.random((n_q, L)) < 0.5).astype(np.uint8)
    db, q = db_from_bytes(ctx, refs), pack_rows(ctx, Q)
    w = oracle.counts(refs, Q, oracle.MIXTURE)
    t = L if hits else -1
    for cap in {max(hits, 1), hits + 5000}:
        got = [x.cpu().numpy() for x in ctx.compare_threshold(db, q, oracle.MIXTURE, t, cap=cap)]
        assert all(np.array_equal(a, b) for a, b in zip(got, oracle.threshold(w, np.full(n_q, t, np.int32))))
    if hits > 1:  # one too many for the caller's buffers: the total comes back
        from paper_1707_00516_amd import FID_EOVERFLOW, fid_compare_threshold, fid_threshold_workspace_bytes
        cap = hits - 1
        thr = torch.full((n_q,), t, dtype=torch.int32, device="cuda")
        ws = torch.empty(fid_threshold_workspace_bytes(db.handle, n_q, cap), dtype=torch.uint8, device="cuda")
        offs, idx = (torch.empty(n, dtype=torch.int64, device="cuda") for n in (n_q + 1, cap))
        cnt = torch.empty(cap, dtype=torch.int32, device="cuda")
        with pytest.raises(FidError) as e:
            fid_compare_threshold(ctx.handle, db.handle, q.data_ptr(), n_q, oracle.MIXTURE, thr.data_ptr(),
                                  ws.data_ptr(), ws.numel(), cap, offs.data_ptr(), idx.data_ptr(), cnt.data_ptr())
        assert e.value.status == FID_EOVERFLOW and e.value.needed == hits
    db.close()
