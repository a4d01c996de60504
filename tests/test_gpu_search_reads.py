"""The search kernel of batches in input order at the sizes where it changes
its ways: one read to several chunks, chunk sizes from 1 to 64 reads, queues
of set-aside reads from one (searched by a whole wave) to full, reads around
a word, a piece and the staging area, reads of up to 1024 bases and one too
long, non-bases at a piece's edges, texts with and without a prefix table
whose brackets hold many rows.  Results are integers: equal to the oracle's."""
import numpy as np
import pytest

import paper_1303_3692_amd as S
from oracle import oracle

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

LENGTHS = [0, 1, 4, 13, 14, 15, 16, 17, 31, 32, 33, 63, 64, 65, 95, 97, 128, 159, 160, 161, 176, 200, 320, 321, 500,
           1008, 1023, 1024]
COUNTS = [1, 2, 3, 5, 8, 9, 16, 17, 31, 32, 33, 63, 64, 65, 130, 700]


def text_of(kind, n, rng):
    t = rng.integers(0, 4, n)
    if kind == "tandem":  # half of it short tandem arrays
        for at in range(0, n - 400, 800):
            u = int(rng.integers(1, 6))
            t[at:at + 400] = np.tile(rng.integers(0, 4, u), 400 // u + 1)[:400]
    elif kind == "copies":  # copies of one element with a few changes
        element = rng.integers(0, 4, 300)
        for at in range(0, n - 300, 600):
            t[at:at + 300] = np.where(rng.random(300) < 0.05, rng.integers(0, 4, 300), element)
    return np.frombuffer(b"ACGT", dtype=np.uint8)[t]


def reads_of(text, rng):
    """700 reads of every length in LENGTHS: copies, copies with changes or non-bases, and unrelated ones."""
    out = []
    for i in range(COUNTS[-1]):
        m = LENGTHS[i % len(LENGTHS)] if i < 400 else int(rng.integers(1, 320))
        r = rng.choice(np.frombuffer(b"ACGT", dtype=np.uint8), m)
        if i % 5 and m <= len(text):
            p = int(rng.integers(0, len(text) - m + 1))
            r = text[p:p + m].copy()
            if i % 5 > 2 and m:
                for at in rng.integers(0, m, 1 + m // 200):
                    r[at] = rng.choice(np.frombuffer(b"ACGTNacgt\x00", dtype=np.uint8))
            if i % 35 == 1 and m > 16:
                r[[15, 16][i % 2]] = ord("N")
        out.append(r)
    order = rng.permutation(len(out))
    return [out[i] for i in order]


@pytest.mark.parametrize("kind,n", [("iid", 3_000), ("tandem", 3_900), ("iid", 60_000), ("tandem", 50_000),
                                    ("copies", 200_000)])
def test_edges_of_the_search_kernel(kind, n):
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    print("case:", kind, n, flush=True)
    rng = np.random.default_rng(n)
    text = text_of(kind, n, rng)
    reads = reads_of(text, rng)
    sa = oracle.sa_build(text)
    d = S.sa_build_device(text, 0)
    dev = torch.device("cuda:0")
    for count in COUNTS:
        some = reads[:count]
        lead = count % 16  # where the batch starts in its buffer
        data = np.concatenate([np.full(lead, ord("C"), np.uint8), *some, np.full(1, ord("A"), np.uint8)])
        offs = lead + np.concatenate([[0], np.cumsum([len(r) for r in some])]).astype(np.int64)
        want = oracle.match(text, sa, data, offs)
        d_reads, d_offs = torch.from_numpy(data).to(dev), torch.from_numpy(offs).to(dev)
        for kw in ({}, dict(defer=0), dict(sort=0), dict(sort=0, prefix_table=0), dict(sort=0, block=1024, blocks_per_cu=1)):
            out = torch.full((count, 4), -7, dtype=torch.int32, device=dev)
            S.match_batch_dev(d, d_reads, d_offs, out, config=S.cfg(d, **kw))
            torch.cuda.synchronize()
            assert (out.cpu().numpy() == want).all(), f"{count} reads, {kw}"


def test_reads_out_of_range_and_out_of_order():
    """A read of 1025 bases and offsets that go back (a negative length, then
    reads that lie before it) among ordinary reads."""
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    rng = np.random.default_rng(5)
    text = text_of("copies", 40_000, rng)
    lengths = [100, 1025, 90, -300, 64, 33, 0, 1024, 20]
    offs = 400 + np.concatenate([[0], np.cumsum(lengths)]).astype(np.int64)
    data = rng.choice(text, 4000)
    data[500:900] = text[700:1100]
    d = S.sa_build_device(text, 0)
    dev = torch.device("cuda:0")
    out = torch.full((len(lengths), 4), -7, dtype=torch.int32, device=dev)
    S.match_batch_dev(d, torch.from_numpy(data).to(dev), torch.from_numpy(offs).to(dev), out)
    torch.cuda.synchronize()
    got, sa = out.cpu().numpy(), oracle.sa_build(text)
    for i, m in enumerate(lengths):
        if m < 0 or m > S.SA_MAX_READ:
            assert tuple(got[i]) == (0, 0, 0, S.SA_HIT_TOOLONG)
        else:
            want = oracle.match(text, sa, data[offs[i]:offs[i + 1]], np.array([0, m], dtype=np.int64))
            assert (got[i] == want[0]).all(), (i, m)


@pytest.mark.parametrize("kind,n", [("copies", 60_000), ("tandem", 40_000), ("iid", 3_500)])
def test_long_reads_in_full_chunks(kind, n):
    """Chunks of 64 (and 16) reads of 20-1024 bases, which are staged by their
    first pieces first: reads settled there, reads that match just up to, up to
    and past what was staged, and non-bases on either side of it."""
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    print("case: long reads,", kind, n, flush=True)
    rng = np.random.default_rng(n)
    text = text_of(kind, n, rng)
    count = 33_000
    lengths = rng.choice([20, 100, 161, 320, 321, 400, 700, 1023, 1024], count)
    offs = 5 + np.concatenate([[0], np.cumsum(lengths)]).astype(np.int64)
    start = rng.integers(0, n - 1024, count)
    data = np.full(int(offs[-1]) + 1, ord("A"), np.uint8)
    owner = np.repeat(np.arange(count), lengths)
    within = np.arange(int(offs[-1]) - 5) - (offs[:-1] - 5)[owner]
    data[5:-1] = text[start[owner] + within]
    for i in np.nonzero(rng.random(count) < 0.7)[0]:  # a change, a non-base, or neither
        at = int(rng.choice([0, 5, 15, 100, 158, 159, 160, 161, 170, 175, 176, 177, 300, 351, 352, 353, 900]))
        if at < lengths[i]:
            data[offs[i] + at] = rng.choice(np.frombuffer(b"ACGTNn", dtype=np.uint8))
    for i in np.nonzero(rng.random(count) < 0.2)[0]:  # unrelated
        data[offs[i]:offs[i + 1]] = rng.choice(np.frombuffer(b"ACGT", dtype=np.uint8), lengths[i])
    want = oracle.match(text, oracle.sa_build(text), data, offs)
    d = S.sa_build_device(text, 0)
    dev = torch.device("cuda:0")
    d_reads, d_offs = torch.from_numpy(data).to(dev), torch.from_numpy(offs).to(dev)
    for some in (count, 9_001):
        for kw in (dict(block=256, blocks_per_cu=1), dict(block=256, blocks_per_cu=1, defer=0),
                   dict(block=256, blocks_per_cu=1, sort=0, prefix_table=0), {}):
            out = torch.full((some, 4), -7, dtype=torch.int32, device=dev)
            S.match_batch_dev(d, d_reads, d_offs, out, nreads=some, config=S.cfg(d, **kw))
            torch.cuda.synchronize()
            assert (out.cpu().numpy() == want[:some]).all(), f"{some} reads, {kw}"
