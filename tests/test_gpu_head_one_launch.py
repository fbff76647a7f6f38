"""The one-launch head kernel, which calls take while TFE_HEAD_WAIT_LIMIT is
set, against the two launches that they take otherwise: ids bit-exact,
probabilities within 1e-5 relative (the denominators are added up in
different orders)."""
import numpy as np
import pytest
import torch

from paper_2607_07388_amd import tfe

from .test_gpu_head_fused import gaussian, one_launch, small_ints

pytestmark = pytest.mark.gpu

WAIT = str(1 << 20)  # polls, about a second: the waits end long before


@pytest.mark.parametrize("V,D,B,K", [
    (151936, 1024, 64, 128), (151936, 1024, 1, 1), (40000, 512, 13, 256), (3001, 256, 5, 17),
    (300, 512, 17, 200)])
def test_one_launch_matches_two(monkeypatch, V, D, B, K):
    w, h = gaussian(V + K, V, D, B)
    head = tfe.tfe_head_create(w, V, D, B, K)
    try:
        want = one_launch(head, h, B, K)  # two launches
        for _ in range(3):
            monkeypatch.setenv("TFE_HEAD_WAIT_LIMIT", WAIT)
            ids, prob = one_launch(head, h, B, K)
            monkeypatch.delenv("TFE_HEAD_WAIT_LIMIT")
            np.testing.assert_array_equal(ids, want[0])
            np.testing.assert_allclose(prob, want[1], rtol=1e-5, atol=1e-37)
            again = one_launch(head, h, B, K)
            np.testing.assert_array_equal(again[0], want[0])
        assert tfe.tfe_head_last_fault(head) == 0
    finally:
        tfe.tfe_head_free(head)


def test_one_launch_heavy_ties(monkeypatch):
    V, D, B, K = 151936, 256, 64, 128
    w, h = small_ints(4, V, D, B, 0, 2)
    head = tfe.tfe_head_create(w, V, D, B, K)
    try:
        want = one_launch(head, h, B, K)
        monkeypatch.setenv("TFE_HEAD_WAIT_LIMIT", WAIT)
        ids, prob = one_launch(head, h, B, K)
        np.testing.assert_array_equal(ids, want[0])
        np.testing.assert_allclose(prob, want[1], rtol=1e-5, atol=1e-37)
    finally:
        tfe.tfe_head_free(head)


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


def test_calls_of_one_head_on_two_streams(monkeypatch):
    """Calls of one head alternate between two streams without
    synchronisation; each waits on the device for the one before."""
    V, D, B, K = 60000, 512, 64, 32
    w, h1 = gaussian(21, V, D, B)
    h2 = torch.flip(h1, [0]).contiguous()
    head = tfe.tfe_head_create(w, V, D, B, K)
    streams = torch.cuda.Stream(), torch.cuda.Stream()
    try:
        want = [one_launch(head, h, B, K) for h in (h1, h2)]
        outs = []
        for i in range(24):
            ids = torch.empty((B, K), dtype=torch.int32, device="cuda")
            prob = torch.empty((B, K), dtype=torch.float32, device="cuda")
            outs.append((ids, prob))
        torch.cuda.synchronize()
        for i, (ids, prob) in enumerate(outs):
            tfe.tfe_head_topk(head, (h1, h2)[i & 1], B, K, ids, prob, streams[i & 1])
        torch.cuda.synchronize()
        for i, (ids, prob) in enumerate(outs):
            np.testing.assert_array_equal(ids.cpu().numpy(), want[i & 1][0])
            np.testing.assert_array_equal(prob.cpu().numpy(), want[i & 1][1])
    finally:
        tfe.tfe_head_free(head)
