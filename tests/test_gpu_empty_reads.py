"""Batches with empty reads among the others, against the oracle: the search
kernel stages the reads around them in one piece."""
import numpy as np
import pytest

import paper_1303_3692_amd as S
from oracle import oracle

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

LETTERS = np.frombuffer(b"ACGT", dtype=np.uint8)


def lengths(kind, count, rng):
    at = np.arange(count)
    m = rng.integers(20, 160, count)
    if kind == "every second":
        m[::2] = 0
    elif kind == "runs":
        m[(at // 7) % 2 == 1] = 0
    elif kind == "nearly all":
        m[at % 61 != 60] = 0
    elif kind == "ends":
        m[:70] = 0
        m[-70:] = 0
    elif kind == "long":  # chunks that take several turns
        m = rng.integers(300, 1025, count)
        m[at % 3 == 1] = 0
    elif kind == "too long":
        m[at % 3 == 1] = 0
        m[at % 5 == 2] = 1025 + at[at % 5 == 2] % 3
    elif kind == "one base":
        m = at % 2
    return m


@pytest.mark.parametrize("kind", ["every second", "runs", "nearly all", "ends", "long", "too long", "one base"])
@pytest.mark.parametrize("n,count", [(3_000, 20_001), (60_000, 300), (60_000, 20_001), (60_000, 500_001)])
def test_empty_reads_among_others(kind, n, count):
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    print("case: empty reads", kind, n, count, flush=True)
    rng = np.random.default_rng(count)
    text = LETTERS[rng.integers(0, 4, n)]
    m = lengths(kind, count, rng)
    offs = np.zeros(count + 1, np.int64)
    np.cumsum(m, out=offs[1:])
    start = rng.integers(0, n - 1100, count)
    owner = np.repeat(np.arange(count), m)
    data = text[np.arange(offs[-1]) - offs[owner] + start[owner]]
    change = rng.random(len(data)) < 0.005
    data[change] = LETTERS[rng.integers(0, 4, int(change.sum()))]
    d = S.sa_build_device(text, 0)
    d_reads, d_offs = torch.from_numpy(data).cuda(), torch.from_numpy(offs).cuda()
    take = np.unique(np.concatenate([np.arange(min(count, 700)), rng.integers(0, count, 700), np.arange(count - 70, count)]))
    whole = take[m[take] <= S.SA_MAX_READ]
    some = np.zeros(len(whole) + 1, np.int64)
    np.cumsum(m[whole], out=some[1:])
    picked = np.concatenate([data[offs[i]:offs[i + 1]] for i in whole])
    want = oracle.match(text, oracle.sa_build(text), picked, some)
    outs = []
    for kw in ({}, {"prefix_table": 0, "sort": 0}, {"defer": 0}):
        out = torch.full((count, 4), -7, dtype=torch.int32, device="cuda")
        S.match_batch_dev(d, d_reads, d_offs, out, config=S.cfg(d, **kw))
        torch.cuda.synchronize()
        outs.append(out)
        got = out.cpu().numpy()
        assert (got[whole, :3] == want[:, :3]).all() and ((got[whole, 3] & 1) == want[:, 3]).all()
        assert (got[m > S.SA_MAX_READ] == [0, 0, 0, S.SA_HIT_TOOLONG]).all()
        assert (got[m == 0] == [0, n, 0, S.SA_HIT_EXACT]).all()
    assert torch.equal(outs[0], outs[1]) and torch.equal(outs[0], outs[2])
