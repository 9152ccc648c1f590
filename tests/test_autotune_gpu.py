"""The autotuner times each plan of its sample batch once: fp4 item lengths beyond what a batch of that size uses give
the same plan, between which timing noise must not choose."""
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


@pytest.mark.parametrize("candidates,plans", [((32, 64, 128, 256, 512), 1), ((1, 2, 512, 256), 3)])
def test_equal_plans_are_timed_once(ctx, candidates, plans, n=200_000, L=64):
    from paper_1707_00516_amd import autotune, fid_row_words
    log(f"autotune candidates {candidates}")
    g = torch.Generator(device="cuda").manual_seed(n)
    rw = fid_row_words(L)

    def rows(m):
        x = torch.randint(-2**63, 2**63 - 1, (m, rw), generator=g, device="cuda", dtype=torch.int64)
        x[:, 1:] = 0
        return x

    db = ctx.build_db(rows(n), L)
    table, report = autotune.tune(ctx, {L: db}, lambda L, r_lo, r_hi, n_q, mode, row0: rows(n_q), k=8, n_jobs=4, reps=1,
                                  q_candidates=(16,), block_candidates=(64,), fp4_tile_candidates=candidates,
                                  log=lambda s: None)
    timed = [key for key in report if "fp4:" in key]
    assert len(timed) == plans, timed
    assert [r[:3] for r in table] == [(L, 16, 64)] and table[0][3] in (0, 1, 2)
    ctx.sync()
    db.close()
