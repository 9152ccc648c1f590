"""Which kernels a top-k call takes -- all counts and a selection, or the list
scan; popcount or fp4 -- follows from its sizes and from the workspace it is
given, and changes nothing in the result: around the lengths and count blocks
where the routes change, with the workspace of the fastest route, with one too
small for it, with the one of another number of queries, without any, and with a
caller's bound.  Reference: every count from the popcount scan, sorted."""
import numpy as np
import pytest

from gpu_harness import log

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


@pytest.mark.parametrize("n,L,n_q", [
    (8192, 8192, 31), (8192, 8192, 32), (8193, 3000, 43), (8193, 3000, 44), (16384, 2048, 31), (16384, 2048, 32),
    (16385, 2048, 15), (16385, 2048, 16), (32768, 1024, 32), (32769, 1024, 31), (65536, 300, 54), (65536, 300, 55),
    (65537, 300, 31), (65537, 300, 32), (513, 2048, 300), (2000, 1024, 600), (40_000, 100, 300), (131072, 64, 3), (131073, 64, 3), (131072, 64, 127), (262144, 64, 200), (262144, 64, 201),
    (262145, 64, 200), (262144, 2048, 5), (262144, 2048, 6), (262145, 2048, 11), (262145, 2048, 12), (33000, 5000, 2),
    (33000, 5000, 1), (540_000, 300, 64), (400_001, 1000, 150), (1_200_000, 100, 17)])
def test_routes_agree(ctx, n, L, n_q, k=5):
    from paper_1707_00516_amd import (FID_BACKEND_AUTO, FID_BACKEND_POPCOUNT, FID_ENOMEM, FidError,
                                      fid_compare_topk, fid_compare_topk_bounded, fid_compare_topk_noalloc,
                                      fid_ctx_set_backend, fid_row_words, fid_topk_mixed_workspace_bytes,
                                      fid_topk_workspace_bytes)
    log(f"routes n={n} L={L} n_q={n_q}")
    rw = fid_row_words(L)
    g = torch.Generator(device="cuda").manual_seed(n + L + n_q)
    bits = torch.randint(-2**63, 2**63 - 1, (n + n_q, rw), generator=g, device="cuda", dtype=torch.int64)
    live = np.zeros(rw * 64, np.uint8)
    live[:L] = 1
    bits &= torch.from_numpy(np.packbits(live, bitorder="little").view(np.int64)).cuda()
    bits[100:n:7] = bits[5]  # equal counts
    db, q = ctx.build_db(bits[:n].contiguous(), L), bits[n:].contiguous()
    want = {}
    fid_ctx_set_backend(ctx.handle, FID_BACKEND_POPCOUNT)
    ids = torch.arange(n, device="cuda")
    for m in (0, 1):
        keys = torch.cat([((c.long() << 40) | ids).topk(k, largest=False).values
                          for c in ctx.compare_full(db, q, m).split(16)])
        want[m] = (keys >> 40).int(), keys & ((1 << 40) - 1)
    fid_ctx_set_backend(ctx.handle, FID_BACKEND_AUTO)
    cnt = torch.empty((n_q, k), dtype=torch.int32, device="cuda")
    idx = torch.empty((n_q, k), dtype=torch.int64, device="cuda")

    def check(m, what):
        ctx.sync()
        assert torch.equal(cnt, want[m][0]) and torch.equal(idx, want[m][1]), what
        cnt.fill_(-1), idx.fill_(-1)

    torch.cuda.synchronize()
    full = fid_topk_workspace_bytes(ctx.handle, db.handle, n_q, k)
    sizes = {full, full - 256, n_q * n * 4 - 256, fid_topk_workspace_bytes(ctx.handle, db.handle, 4 * n_q, k)}
    ran = 0
    for b in sorted(x for x in sizes if x > 0):
        ws = torch.empty(b, dtype=torch.uint8, device="cuda")
        for m in (0, 1):
            try:
                fid_compare_topk(ctx.handle, db.handle, q.data_ptr(), n_q, m, k, ws.data_ptr(), b, cnt.data_ptr(),
                                 idx.data_ptr())
            except FidError as e:
                assert e.status == FID_ENOMEM and b < full
                continue
            check(m, f"workspace {b} of {full}")
            ran += 1
    assert ran >= 2
    for m in (0, 1):
        fid_compare_topk_noalloc(ctx.handle, db.handle, q.data_ptr(), n_q, m, k, cnt.data_ptr(), idx.data_ptr())
        check(m, "noalloc")
        modes = torch.full((n_q,), m, dtype=torch.int32, device="cuda")
        bound = torch.full((n_q,), -1, dtype=torch.int32, device="cuda")
        b = fid_topk_mixed_workspace_bytes(ctx.handle, db.handle, 0, n, n_q, k)
        ws = torch.empty(b, dtype=torch.uint8, device="cuda")
        torch.cuda.synchronize()
        fid_compare_topk_bounded(ctx.handle, db.handle, 0, n, q.data_ptr(), modes.data_ptr(), n_q, k, bound.data_ptr(),
                                 True, ws.data_ptr(), b, cnt.data_ptr(), idx.data_ptr())
        check(m, "bounded")
    db.close()
