"""The whole-network plan's ranking and gather where words of 64 filters can go wrong: one filter, a word less one, a full
word, one more, 1024 and the most filters a ranked layer may have; one survivor, most and all; many equal scores, zero
scores, infinities.  Weights are small whole numbers, so scores are exact; two layers, the second gathered by the first
one's kept list, against numpy bit for bit."""
import numpy as np
import pytest
import torch

from paper_2207_01260_amd import binding as B

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("c", [1, 7, 63, 64, 65, 130, 1000, 1024, 1025, 4095, 4096])
def test_plan_ranking_and_gather_at_word_edges(c):
    for keep in sorted({1, max(1, c // 2), max(1, c - 1), c}):
        print("plan ranking", c, keep, flush=True)
        rng = np.random.default_rng(1000 * c + keep)
        w = rng.integers(-3, 4, (c, 3, 1, 1)).astype(np.float32)   # ten different scores: nearly all are ties
        w[rng.integers(0, c, 1 + c // 9)] = 0.0
        if c > 64:
            w[c - 2, 1] = np.inf
        v = rng.integers(-9, 10, (70, c, 1, 2)).astype(np.float32)
        order = np.lexsort((np.arange(c), -np.abs(w.astype(np.float64)).sum((1, 2, 3))))
        kept = np.sort(order[:keep])
        second = np.sort(np.lexsort((np.arange(70), -np.abs(v.astype(np.float64)).sum((1, 2, 3))))[:66])
        plan = B.PrunePlan([{"w": torch.from_numpy(w).cuda(), "keep": keep, "rows_from": 0, "cols_from": -1},
                            {"w": torch.from_numpy(v).cuda(), "keep": 66, "rows_from": 1, "cols_from": 0}], 1e-5)
        for rep in range(2):
            plan.run()
            torch.cuda.synchronize()
            assert np.array_equal(plan.kept[0].cpu().numpy(), kept), (c, keep, rep)
            assert np.array_equal(plan.kept[1].cpu().numpy(), second), (c, keep, rep)
            assert np.array_equal(plan.w_out[0].cpu().numpy(), w[kept]), (c, keep, rep)
            assert np.array_equal(plan.w_out[1].cpu().numpy(), v[second][:, kept]), (c, keep, rep)
        plan.close()


def test_runs_that_overlap_while_weights_change_stay_in_bounds():
    """Two streams run one plan while a third swaps its weights: results of those runs are not defined, but every kept index is a
    filter and every gathered value one of the sources' (all powers of two here), and a run by itself afterwards is right."""
    c, keep = 1024, 500
    rng = np.random.default_rng(7)
    sources = [2.0 ** rng.integers(-8, 9, (c, 9, 1, 1)).astype(np.float32) for _ in range(2)]
    v = 2.0 ** rng.integers(-8, 9, (70, c, 1, 2)).astype(np.float32)
    dev = [torch.from_numpy(q).cuda() for q in sources]
    w = dev[0].clone()
    plan = B.PrunePlan([{"w": w, "keep": keep, "rows_from": 0, "cols_from": -1},
                        {"w": torch.from_numpy(v).cuda(), "keep": 66, "rows_from": 1, "cols_from": 0}], 1e-5)
    streams = [torch.cuda.Stream() for _ in range(3)]
    torch.cuda.synchronize()
    for rep in range(50):
        for k, s in enumerate(streams):
            with torch.cuda.stream(s):
                if k == 2:
                    w.copy_(dev[rep & 1])
                else:
                    plan.run()
        if rep % 10 == 9:
            torch.cuda.synchronize()
            print("overlapping plan runs", rep, flush=True)
            kept = plan.kept[0].cpu().numpy()
            assert kept.min() >= 0 and kept.max() < c
            for got in (plan.w_out[0], plan.w_out[1]):
                assert np.isin(got.cpu().numpy(), 2.0 ** np.arange(-8, 9)).all()
    w.copy_(dev[1])
    torch.cuda.synchronize()
    plan.run()
    torch.cuda.synchronize()
    order = np.lexsort((np.arange(c), -sources[1].astype(np.float64).sum((1, 2, 3))))
    kept = np.sort(order[:keep])
    second = np.sort(np.lexsort((np.arange(70), -v.astype(np.float64).sum((1, 2, 3))))[:66])
    assert np.array_equal(plan.kept[0].cpu().numpy(), kept)
    assert np.array_equal(plan.w_out[0].cpu().numpy(), sources[1][kept])
    assert np.array_equal(plan.w_out[1].cpu().numpy(), v[second][:, kept])
    plan.close()
