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
