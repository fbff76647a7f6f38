"""The one-launch head kernel, which every call that fits it takes while
TFE_HEAD_WAIT_LIMIT is set, against the two launches (tfe_head_topk_noalloc):
ids bit-exact, probabilities within 1e-5 relative (the denominators are added
up in different orders); calls of one head by both routes in turn; and that
a call takes the faster route."""
import numpy as np
import pytest
import torch

from paper_2607_07388_amd import tfe

from . import harness as H
from .test_gpu_head_fused import WAIT, gaussian, one_launch, small_ints, two_launch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("V,D,B,K", [
    (151936, 1024, 64, 128), (151936, 1024, 1, 1), (40000, 512, 13, 256), (3001, 256, 5, 17),
    (300, 512, 17, 200)])
def test_one_launch_matches_two(monkeypatch, V, D, B, K):
    w, h = gaussian(V + K, V, D, B)
    head = tfe.tfe_head_create(w, V, D, B, K)
    try:
        want = two_launch(w, V, D, h, B, K)
        for _ in range(3):
            monkeypatch.setenv("TFE_HEAD_WAIT_LIMIT", WAIT)
            ids, prob = one_launch(head, h, B, K)
            monkeypatch.delenv("TFE_HEAD_WAIT_LIMIT")
            np.testing.assert_array_equal(ids, want[0])
            np.testing.assert_allclose(prob, want[1], rtol=1e-5, atol=1e-37)
            again = one_launch(head, h, B, K)  # by its own route
            np.testing.assert_array_equal(again[0], want[0])
        assert tfe.tfe_head_last_fault(head) == 0
    finally:
        tfe.tfe_head_free(head)


def test_one_launch_heavy_ties(monkeypatch):
    V, D, B, K = 151936, 256, 64, 128
    w, h = small_ints(4, V, D, B, 0, 2)
    head = tfe.tfe_head_create(w, V, D, B, K)
    try:
        want = two_launch(w, V, D, h, B, K)
        monkeypatch.setenv("TFE_HEAD_WAIT_LIMIT", WAIT)
        ids, prob = one_launch(head, h, B, K)
        np.testing.assert_array_equal(ids, want[0])
        np.testing.assert_allclose(prob, want[1], rtol=1e-5, atol=1e-37)
    finally:
        tfe.tfe_head_free(head)


@pytest.mark.parametrize("V,D,B,K", [(1000, 256, 1, 64), (4000, 256, 1, 256), (4000, 1024, 64, 256),
                                     (16000, 512, 16, 128), (151936, 512, 17, 256)])
def test_the_faster_route_is_taken(monkeypatch, V, D, B, K):
    """A call takes at most 1.2 times what it takes by one launch, and 1.4 times
    what the no-allocation entry point's two launches take (which record no
    event for the next call)."""
    w, h = gaussian(5, V, D, B)
    head = tfe.tfe_head_create(w, V, D, B, K)
    ids = torch.empty((B, K), dtype=torch.int32, device="cuda")
    prob = torch.empty((B, K), dtype=torch.float32, device="cuda")

    def took(call):
        best = float("inf")
        for _ in range(6):
            e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            torch.cuda.synchronize()
            e0.record()
            for _ in range(40):
                call()
            e1.record()
            torch.cuda.synchronize()
            best = min(best, e0.elapsed_time(e1) * 1000 / 40)
        return best

    try:
        own = took(lambda: tfe.tfe_head_topk(head, h, B, K, ids, prob, H.cur_stream()))
        two = took(lambda: tfe.tfe_head_topk_noalloc(w, V, D, h, B, K, ids, prob, H.cur_stream()))
        monkeypatch.setenv("TFE_HEAD_WAIT_LIMIT", WAIT)
        one = took(lambda: tfe.tfe_head_topk(head, h, B, K, ids, prob, H.cur_stream()))
    finally:
        tfe.tfe_head_free(head)
    assert own < 1.2 * one and own < 1.4 * two, (own, one, two)


def test_faults_are_numbered_over_the_calls_that_fit_one_launch(monkeypatch):
    """Calls of at most 64 rows count, by whichever route; larger ones do not
    (they never took one launch)."""
    V, D, B, K = 9000, 256, 100, 16
    w, h = gaussian(33, V, D, B)
    head = tfe.tfe_head_create(w, V, D, B, K)

    def gives_up(rows):
        monkeypatch.setenv("TFE_HEAD_WAIT_LIMIT", "0")
        ids, prob = one_launch(head, h, rows, K)
        monkeypatch.delenv("TFE_HEAD_WAIT_LIMIT")
        return np.all(ids == -1) and np.all(prob == 0)

    try:
        want = one_launch(head, h, B, K)[0]                     # two launches, not counted
        assert gives_up(8)                                      # 1
        assert tfe.tfe_head_last_fault(head) == 1
        for rows in (100, 65):
            np.testing.assert_array_equal(one_launch(head, h, rows, K)[0], want[:rows])
        assert tfe.tfe_head_last_fault(head) == 1
        np.testing.assert_array_equal(one_launch(head, h, 8, K)[0], want[:8])  # 2: two launches
        one_launch(head, h, 70, K)
        assert gives_up(64)                                     # 3
        assert tfe.tfe_head_last_fault(head) == 3
        assert not gives_up(100)                                # never one launch
        assert tfe.tfe_head_last_fault(head) == 3
    finally:
        tfe.tfe_head_free(head)


def test_calls_of_one_head_on_two_streams():
    """Calls of one head alternate between two streams without
    synchronisation, and between the routes (64 rows by one launch, 8 by two);
    each waits on the device for the one before."""
    V, D, K = 151936, 512, 32
    w, h1 = gaussian(21, V, D, 64)
    h2 = torch.flip(h1, [0])[:8].contiguous()
    rows = (h1, 64), (h2, 8)
    head = tfe.tfe_head_create(w, V, D, 64, K)
    streams = torch.cuda.Stream(), torch.cuda.Stream()
    try:
        want = [two_launch(w, V, D, h, B, K) for h, B in rows]
        outs = []
        for i in range(36):
            # Both routes follow each other on one stream and across the two.
            (h, B), s = rows[i & 1], streams[(i // 3) & 1]
            outs.append((i & 1, torch.empty((B, K), dtype=torch.int32, device="cuda"),
                         torch.empty((B, K), dtype=torch.float32, device="cuda"), h, B, s))
        torch.cuda.synchronize()
        for _, ids, prob, h, B, s in outs:
            tfe.tfe_head_topk(head, h, B, K, ids, prob, s)
        torch.cuda.synchronize()
        for r, ids, prob, _, _, _ in outs:
            np.testing.assert_array_equal(ids.cpu().numpy(), want[r][0])
            np.testing.assert_allclose(prob.cpu().numpy(), want[r][1], rtol=1e-5, atol=1e-37)
        assert tfe.tfe_head_last_fault(head) == 0
    finally:
        tfe.tfe_head_free(head)
