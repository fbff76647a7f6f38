"""Count tables of tfe_ngram_top that hold fewer distinct n-grams than they are
given: slices that are regrouped and counted part by part, parts that are too
large all the same, merges of slices in parts.  Results are compared with the
oracle (tuples and counts bit-exact), and the time of long streams of distinct
n-grams with the time of shorter ones.

The windows that meet in one table are chosen with the window split and the
hash of the count tables, restated here: a stream of up to 2^18 x 16384 windows
has 512 partitions for these sizes, slices hold 16384 windows, tables 16384
entries (n = 2) or 8192 (n > 2), and the low bits of the hash pick a remainder's
part."""
import time

import numpy as np
import pytest
import torch

from paper_2607_07388_amd import tfe

from . import harness as H
from .test_gpu_build import check

pytestmark = pytest.mark.gpu

TOK = (1 << 18) - 1
LOW = 18 - 9  # bits of the scrambled oldest token below the partition number
MIX = 0x2E5B5
U = np.uint64
M32 = U(0xFFFFFFFF)


def tail_hash(x):
    """Of the tokens after the oldest (columns 1..3 of x, 0 where absent)."""
    mul24 = lambda a, b: ((a & U(0xFFFFFF)) * U(b)) & M32
    h = (mul24(x[:, 1], 0xC2B2AD) + mul24(x[:, 2], 0x9E3779) + mul24(x[:, 3], 0x85EBCB)) & M32
    h ^= h >> U(16)
    return mul24(h, 0xD35A2D) >> U(14)


def windows_of(part, rem, n):
    """The n-token windows of partition `part` with these remainders."""
    x = np.zeros((rem.size, 4), np.uint64)
    r = rem.astype(np.uint64)
    for q in range(n - 1, 0, -1):
        x[:, q] = r & U(TOK)
        r = r >> U(18)
    m = U(part << LOW) | r
    x[:, 0] = ((m ^ tail_hash(x)) * U(pow(MIX, -1, 1 << 18))) & U(TOK)
    # The split gives the partition back.
    assert np.all((((x[:, 0] * U(MIX)) & U(TOK)) ^ tail_hash(x)) >> U(LOW) == U(part))
    return x[:, :n].astype(np.int32)


def unshift(h, s):
    """Inverse of h ^= h >> s on 32 bits."""
    x = h
    for _ in range(32 // s + 1):
        x = h ^ (x >> U(s))
    return x


def unmul(h, m):
    return (h * U(pow(m, -1, 1 << 32))) & M32


def remainders_with_hash(h, n, rng):
    """Distinct remainders whose table hash is one of h (32-bit words)."""
    h = h.astype(np.uint64)
    if n == 2:  # a 32-bit word, of which a remainder has 27 bits
        r = unmul(unshift(unmul(unshift(h, 13), 0x85EBCA77), 15), 0x9E3779B1)
        return np.unique(r[r < U(1 << 27)])
    hi = rng.permutation(1 << min(LOW + 18 * (n - 1) - 32, 20)).astype(np.uint64)[:h.size]
    h = h[:hi.size]
    mixed = unshift(unmul(unshift(h, 13), 0xC2B2AE3D), 15)
    lo = unmul(mixed ^ ((hi * U(0x85EBCA77)) & M32), 0x9E3779B1)
    return np.unique((hi << U(32)) | lo)


def stream(windows, copies, rng):
    """The windows, each `copies` times, in random order, broken apart by -1."""
    w = np.repeat(windows, copies, axis=0)
    w = w[rng.permutation(len(w))]
    return np.concatenate([w, np.full((len(w), 1), -1, np.int32)], axis=1).ravel()


@pytest.mark.parametrize("n,count,twice,heavy", [
    (2, 60000, 0, 1), (3, 60000, 20000, 1), (4, 60000, 20000, 1),  # several slices, all too full; merges too
    (3, 9000, 500, 1), (4, 16000, 0, 1),                # one slice, one table too few
    (2, 16384, 0, 1), (3, 8192, 0, 1), (4, 8192, 0, 1), # a window for every entry
    (3, 7200, 0, 1), (4, 7100, 0, 1),                   # just more and less than 7/8 of the entries
    (3, 9500, 0, 3000), (4, 12000, 0, 4000),            # too many, though the first windows repeat
    (3, 4200, 0, 9000), (4, 5000, 0, 11000),            # not too many
])
def test_distinct_ngrams_of_one_partition(n, count, twice, heavy):
    rng = np.random.default_rng(1000 * n + count)
    rem = rng.choice(1 << min(LOW + 18 * (n - 1), 40), count + 200, replace=False)[:count]
    copies = np.ones(count, np.int64)
    copies[rng.permutation(count)[:twice]] = 2
    copies[0] = heavy
    tok = stream(windows_of(5, rem, n), copies, rng)
    assert tok.size < 512 * 16384 // 2  # 512 partitions, slices of 16384
    check(tok, 1 << 18, n, 3, 2 * count)
    check(tok, 1 << 18, n, 0, 1000)


@pytest.mark.parametrize("n", [2, 3])
def test_remainders_that_share_their_low_hash_bits(n):
    """Every remainder falls into the same part of a regrouped slice, which
    has to be split by further bits."""
    rng = np.random.default_rng(70 + n)
    h = (rng.permutation(1 << 20).astype(np.uint64) << U(12)) | U(0xABC)
    rem = rng.permutation(remainders_with_hash(h, n, rng))[:30000 if n == 2 else 8192]
    if n == 3:  # 13 upper bits only: as many again with another low part
        rem = np.unique(np.concatenate([rem, remainders_with_hash(h[::-1], n, rng)]))
    assert rem.size > (16384 if n == 2 else 8192)
    copies = 1 + (np.arange(rem.size) % 5 == 0)
    check(stream(windows_of(3, rem, n), copies, rng), 1 << 18, n, 0, rem.size)


def test_remainders_of_one_hash():
    """Every remainder has the same home bucket, step and part: the table is
    full for them at a few dozen, and parts are told apart by the remainders'
    own bits."""
    rng = np.random.default_rng(80)
    rem = remainders_with_hash(np.full(9000, 0x12345678), 4, rng)
    assert rem.size == 9000
    copies = 1 + (np.arange(rem.size) % 7 == 0)
    check(stream(windows_of(9, rem, 4), copies, rng), 1 << 18, 4, 0, rem.size)


@pytest.mark.parametrize("n,N", [(2, 1 << 22), (3, 1 << 24), (4, 1 << 24)])
def test_long_streams_keep_the_rate(n, N):
    """Evenly drawn tokens (nearly every window distinct): four times the
    stream takes about four times as long, though its partitions no longer fit
    a table (1.6 times that allowed; tables found full by halving took 12 to
    26 times as long)."""
    top = 50000
    tup = torch.empty((top, n), dtype=torch.int32, device="cuda")
    cnt = torch.empty(top, dtype=torch.int64, device="cuda")
    g = torch.Generator(device="cuda")
    g.manual_seed(n)
    tok = torch.randint(0, 1 << 18, (4 * N,), generator=g, device="cuda", dtype=torch.int32)

    def best(size):
        t = []
        for _ in range(6):
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            assert tfe.tfe_ngram_top(tok, size, 1 << 18, n, 0, top, tup, cnt, H.cur_stream()) == top
            t.append(time.perf_counter() - t0)
        return min(t)

    short, long = best(N), best(4 * N)
    tfe.tfe_ngram_release()
    assert long < 1.6 * 4 * short, (short, long)
