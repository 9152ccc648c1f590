"""Threshold hits appended by a tick's top-k scan (whole-database ticks over a
range that the list scan takes, on the matrix cores): requests with and
without thresholds, of one mode and of both, each equal to its own top-k and
threshold call on the popcount scan, bit-exact."""
import numpy as np
import pytest

from gpu_harness import log

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("L,sizes,modes", [(300, (64,), (0,)), (300, (60, 25, 50), (0, 1, 0)), (2100, (20, 13), (1, 1))])
def test_hits_of_the_topk_scan(L, sizes, modes):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1707_00516_amd import FID_BACKEND_POPCOUNT, fid_ctx_set_backend, fid_row_words
    from paper_1707_00516_amd.torch_api import Context, Server
    log(f"server hits L={L} sizes={sizes} modes={modes}")
    n = 270_001  # longer than the ranges whose counts are all written
    ctx, plain = Context(0), Context(0)
    fid_ctx_set_backend(plain.handle, FID_BACKEND_POPCOUNT)
    g = torch.Generator(device="cuda").manual_seed(L + len(sizes))
    rw = fid_row_words(L)
    bits = torch.randint(-2**63, 2**63 - 1, (n + sum(sizes), rw), generator=g, device="cuda", dtype=torch.int64)
    live = np.zeros(rw * 64, np.uint8)
    live[:L] = 1
    bits &= torch.from_numpy(np.packbits(live, bitorder="little").view(np.int64)).cuda()
    db = ctx.build_db(bits[:n].contiguous(), L)
    torch.cuda.synchronize()
    srv = Server(ctx, db, 1 << 30, 4096, 32, 4, 0, 0, 0)
    at, asked = n, []
    for i, (nq, m) in enumerate(zip(sizes, modes)):
        q = bits[at:at + nq].contiguous()
        at += nq
        low = plain.compare_topk(db, q, m, 32)
        plain.sync()
        t = None if i == 1 else int(low[0][:, 20].max().item())
        hits = None if t is None else [x.cpu().numpy() for x in plain.compare_threshold(db, q, m, t)]
        asked.append((q, m, t, [x.cpu().numpy() for x in low], hits))
    tickets = [srv.submit(q, m, thr=None if t is None else np.full(q.shape[0], t, np.int32),
                          hit_cap=0 if t is None else int(hits[0][-1]))
               for q, m, t, _, hits in asked]
    for ticket, (_, _, t, low, hits) in zip(tickets, asked):
        res = srv.wait(ticket, timeout_us=60_000_000)
        assert np.array_equal(res[0], low[0]) and np.array_equal(res[1], low[1])
        if t is not None:
            assert all(np.array_equal(a, b) for a, b in zip(res[3], hits))
    srv.close()
    db.close()
    ctx.close()
    plain.close()
