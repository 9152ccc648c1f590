"""Copy streams of the streamed calls, borrowed from a pool of the device: contexts in several threads stream at once
and one after another, some destroyed in between, each with the oracle's results; and a new context's first streamed
call beside others does not pay for streams of its own."""
import threading
import time

import numpy as np
import pytest

import oracle
from gpu_harness import log, pack_rows

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

L, N, NQ, K, BLOCK, THR = 300, 5000, 6, 8, 700, 60


@pytest.fixture(scope="module")
def world():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1707_00516_amd.torch_api import Context
    ctx = Context(0)
    out = []
    for seed in range(4):
        rng = np.random.default_rng(seed)
        refs = (rng.random((N, L)) < 0.3).astype(np.uint8)
        Q = (rng.random((NQ, L)) < 0.4).astype(np.uint8)
        counts = oracle.counts(refs, Q, oracle.MIXTURE)
        hits = [np.nonzero(c <= THR)[0] for c in counts]
        out.append(dict(rows=pack_rows(ctx, refs).cpu().pin_memory(), q=pack_rows(ctx, Q), counts=counts, hits=hits,
                        topk=oracle.topk(counts, K)))
    ctx.sync()
    yield ctx, out
    ctx.close()


def _stream_all(ctx, w):
    thr = torch.full((NQ,), THR, dtype=torch.int32, device="cuda")
    cnt, idx = ctx.compare_topk_streamed(w["rows"], L, BLOCK, w["q"], oracle.MIXTURE, K)
    offs, hidx, _ = ctx.compare_threshold_streamed(w["rows"], L, BLOCK, w["q"], oracle.MIXTURE, thr)
    full = ctx.compare_full_streamed(w["rows"], L, BLOCK, w["q"], oracle.MIXTURE)
    ctx.sync()
    assert np.array_equal(cnt.cpu().numpy(), w["topk"][0]) and np.array_equal(idx.cpu().numpy(), w["topk"][1])
    assert np.array_equal(full.numpy(), w["counts"])
    offs = offs.cpu().numpy()
    assert np.array_equal(offs, np.concatenate(([0], np.cumsum([len(h) for h in w["hits"]]))))
    assert np.array_equal(hidx.cpu().numpy(), np.concatenate(w["hits"]))


def test_contexts_of_several_threads(world):
    from paper_1707_00516_amd.torch_api import Context
    failed = []

    def work(i):
        try:
            with torch.cuda.stream(torch.cuda.Stream()):
                for rep in range(4):
                    ctx = Context(0)
                    for j in range(3):
                        _stream_all(ctx, world[1][(i + rep + j) % 4])
                    ctx.close()
        except BaseException as e:  # noqa: BLE001  (reported by the test's own thread)
            failed.append((i, repr(e)))

    torch.cuda.synchronize()
    threads = [threading.Thread(target=work, args=(i,)) for i in range(6)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not failed, failed[0]
    _stream_all(world[0], world[1][0])


def test_first_call_of_a_new_context(world):
    """Streams of a context's own cost its first call 3 ms and more each until the process has its four hardware
    queues; a borrowed one costs nothing.  Four new contexts, so that one of them would be the first to need more."""
    from paper_1707_00516_amd.torch_api import Context
    w = world[1][0]

    def call(ctx):
        torch.cuda.synchronize()
        t = time.perf_counter()
        ctx.compare_topk_streamed(w["rows"], L, BLOCK, w["q"], oracle.MIXTURE, K)
        return (time.perf_counter() - t) * 1e3

    for _ in range(4):
        call(world[0])
    later = min(call(world[0]) for _ in range(5))
    new = [Context(0) for _ in range(4)]
    first = [call(c) for c in new]
    log(f"later calls {later:.2f} ms, first calls of new contexts {first}")
    for c in new:
        c.close()
    assert max(first) < later + 2.0
