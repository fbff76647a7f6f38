"""GPU parity of every branch of tfe_ngram_top against the oracle (tuples and
counts bit-exact): partitions counted in one slice and in several, count
tables that fill up and are retried on parts of the remainders, the tie
selection, and the three rankings (one bucket, bucket sort, radix sort)."""
import numpy as np
import pytest
import torch

import oracle
from paper_2607_07388_amd import tfe

from . import harness as H
from .test_gpu_build import check

pytestmark = pytest.mark.gpu


def uniform(seed, N, vocab):
    return np.random.default_rng(seed).integers(0, vocab, N).astype(np.int32)


@pytest.mark.parametrize("n,N,vocab,skip,top", [
    # Up to 512 partitions of 11700 windows, nearly all distinct: 2-grams fill three
    # quarters of a table, 3- and 4-grams (8192 entries) overflow it and retry.
    (2, 6000000, 1 << 18, 0, 3000),
    (3, 5600000, 1 << 18, 0, 3000),
    (4, 5600000, 1 << 18, 7, 3000),
    # Every window asked for: the bucket sort, then records beyond it.
    (3, 1500000, 1 << 17, 100, 1500000),
    (2, 9000000, 1 << 18, 5, 9000000),
    (4, 4600000, 1 << 18, 5, 4600000),
    # Few ranks wanted of many equal counts: the tie selection (about 2^21 windows seen once).
    (1, 500000, 1 << 18, 0, 100),
    (2, 2200000, 1 << 18, 0, 2000),
    (4, 2200000, 1 << 18, 3, 2000),
])
def test_uniform_streams(n, N, vocab, skip, top):
    check(uniform(N + n, N, vocab), vocab, n, skip, top)


@pytest.mark.parametrize("n,prefix,first", [
    (2, [], 1 << 18), (2, [], 512), (3, [7], 1 << 18), (3, [], 512), (3, [7], 512),
    (4, [7], 1 << 18), (4, [7, 9], 1 << 18), (4, [7, 9], 512)])
def test_ties_that_share_their_oldest_tokens(n, prefix, first):
    """1.5M windows, nearly all seen once, whose oldest tokens (and with first = 512
    the high digit of the next) are the same: the tie selection goes through
    one digit to all before the newest token's."""
    rng = np.random.default_rng(first + 10 * n + len(prefix))
    w = rng.integers(0, 1 << 18, (1500000, n + 1)).astype(np.int32)
    w[:, :len(prefix)] = prefix
    w[:, len(prefix)] = rng.integers(0, first, len(w))
    w[:, n] = -1
    key = w[:, n - 2].astype(np.int64) << 18 | w[:, n - 1]  # the tokens that differ, and more
    assert (np.unique(key, return_counts=True)[1] == 1).sum() > (1 << 20) + 4 * 3000
    extra = w[rng.permutation(len(w))[:1000]]  # and some above the ties
    tok = np.concatenate([w, extra, extra]).ravel()
    check(tok, 1 << 18, n, 5, 3000)


@pytest.mark.parametrize("n", [1, 2, 3, 4])
def test_one_ngram_fills_a_partition(n):
    """Half the stream repeats one token: its partition spans several slices,
    whose counts are added up."""
    rng = np.random.default_rng(60 + n)
    tok = rng.integers(0, 3000, 900000).astype(np.int32)
    tok[200000:650000] = 17
    tok[rng.random(tok.size) < 0.001] = -1
    check(tok, 3000, n, 0, 5000)


@pytest.mark.parametrize("shift", [1, 2, 3])
def test_stream_not_16_byte_aligned(shift):
    tok = uniform(70 + shift, 100003, 500)
    dev = torch.from_numpy(np.concatenate([np.zeros(shift, np.int32), tok])).cuda()[shift:]
    assert dev.data_ptr() % 16 == 4 * shift
    for n in (2, 4):
        tup = torch.zeros((1000, n), dtype=torch.int32, device="cuda")
        cnt = torch.zeros((1000,), dtype=torch.int64, device="cuda")
        m = tfe.tfe_ngram_top(dev, tok.size, 500, n, 0, 1000, tup, cnt, H.cur_stream())
        want_t, want_c = oracle.ngram_top(tok, 500, n, 0, 1000)
        np.testing.assert_array_equal(tup[:m].cpu().numpy(), want_t)
        np.testing.assert_array_equal(cnt[:m].cpu().numpy(), want_c)
