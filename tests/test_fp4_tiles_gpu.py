"""The fp4 scan at the edges of its tiles, against the oracle, bit-exact: query
counts around the 16-query blocks and 128-query tiles (and the even split of
the blocks over the tiles), row lengths around the 512-locus groups, the
1024-locus LDS halves and the rows of two halves that stay resident, reference
ranges that cut a 64-reference block at both ends or leave blocks of padding,
queries of both modes in one tile, and a queue of candidates that overflows."""
import numpy as np
import pytest

import gen
import oracle
from gpu_harness import db_from_bytes, log, pack_rows, to_dev

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

N_REFS = 17_001  # longer than a top-k call's seed prefix of 16,384 references


@pytest.fixture(scope="module")
def ctx():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1707_00516_amd import FID_BACKEND_MFMA_FP4, fid_ctx_set_backend
    from paper_1707_00516_amd.torch_api import Context
    c = Context(0)
    fid_ctx_set_backend(c.handle, FID_BACKEND_MFMA_FP4)
    yield c
    c.sync()
    c.close()


@pytest.mark.parametrize("n_q,L", [(1, 512), (16, 1), (17, 513), (33, 1024), (48, 1025), (65, 1536), (97, 2048),
                                   (112, 2049), (113, 2560), (128, 3073), (129, 700), (131, 2048), (200, 4097),
                                   (257, 31)])
def test_fp4_tile_edges(ctx, n_q, L):
    log(f"fp4 tile edges n_q={n_q} L={L}")
    thr = gen.maf_thresholds(900 + L, L, 0.05)
    refs = gen.ref_bytes(900 + L, thr, 0, N_REFS)
    Q = gen.mixtures(900 + L, thr, 0, N_REFS, 0, n_q, 1, 4, 0.005)[0]
    db, q = db_from_bytes(ctx, refs), pack_rows(ctx, Q)
    want = {m: oracle.counts(refs, Q, m) for m in (oracle.MIXTURE, oracle.IDENTITY)}
    for m, w in want.items():
        assert np.array_equal(ctx.compare_full(db, q, m).cpu().numpy(), w)
        t = int(np.partition(w, 40, axis=1)[:, 40].min())
        offs, idx, cnt = ctx.compare_threshold(db, q, m, t)
        wo, wi, wc = oracle.threshold(w, np.full(n_q, t, np.int32))
        assert np.array_equal(offs.cpu().numpy(), wo) and np.array_equal(idx.cpu().numpy(), wi)
        assert np.array_equal(cnt.cpu().numpy(), wc)
        bo, bi, bc, tc, ti = (x.cpu().numpy() for x in ctx.compare_threshold_topk(db, q, m, t, 32))
        wtc, wti = oracle.topk(w, 32)
        assert np.array_equal(bo, wo) and np.array_equal(bi, wi) and np.array_equal(bc, wc)
        assert np.array_equal(tc, wtc) and np.array_equal(ti, wti)
    # a range that starts and ends inside a block, queries of both modes
    modes = (np.arange(n_q) % 3 == 1).astype(np.int32)
    mixed = np.where(modes[:, None] == oracle.IDENTITY, want[oracle.IDENTITY], want[oracle.MIXTURE])
    for lo, hi in ((37, N_REFS - 5), (0, N_REFS - 64)):
        cnt, idx = ctx.compare_topk_mixed(db, lo, hi, q, to_dev(modes), 10)
        wc, wi = oracle.topk(mixed[:, lo:hi], 10)
        assert np.array_equal(cnt.cpu().numpy(), wc) and np.array_equal(idx.cpu().numpy(), wi + lo)
    db.close()


@pytest.mark.parametrize("n_q", [3, 100, 131])
def test_fp4_queue_overflow_with_hits(ctx, n_q):
    """Identical references: every pair is a top-k candidate and a threshold
    hit, so each tile's queue of 64 fills up again and again."""
    log(f"fp4 queue overflow n_q={n_q}")
    L = 300
    rng = np.random.default_rng(n_q)
    refs = np.repeat((rng.random((1, L)) < 0.3).astype(np.uint8), N_REFS, axis=0)
    Q = (rng.random((n_q, L)) < 0.5).astype(np.uint8)
    db, q = db_from_bytes(ctx, refs), pack_rows(ctx, Q)
    for m in (oracle.MIXTURE, oracle.IDENTITY):
        w = oracle.counts(refs, Q, m)
        got = [x.cpu().numpy() for x in ctx.compare_threshold_topk(db, q, m, L, 7, cap=n_q * N_REFS)]
        exp = [*oracle.threshold(w, np.full(n_q, L, np.int32)), *oracle.topk(w, 7)]
        assert all(np.array_equal(a, b) for a, b in zip(got, exp))
    db.close()
