"""Locate calls and batches of several threads on one index."""
import threading

import numpy as np
import pytest

import paper_1303_3692_amd as S

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def index():
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    text = np.random.default_rng(1).choice(np.frombuffer(b"ACGT", dtype=np.uint8), 100_000)
    host = S.sa_build(text)
    return text, host.suffix_array(), S.sa_upload(host, 0)


def test_a_batch_is_enqueued_while_a_locate_waits(index):
    """A locate waits for its stream; a batch that another thread puts on the
    same stream meanwhile is enqueued at once."""
    text, _, d = index
    reads = torch.from_numpy(text[:6000].copy()).cuda()
    offs = torch.arange(101, device="cuda") * 60
    hits = torch.zeros((100, 4), dtype=torch.int32, device="cuda")
    again = torch.full((100, 4), -7, dtype=torch.int32, device="cuda")
    starts = torch.zeros(101, dtype=torch.int64, device="cuda")
    pos = torch.zeros(1000, dtype=torch.int32, device="cuda")
    a = torch.rand((8192, 8192), device="cuda")
    b = torch.empty_like(a)
    stream = torch.cuda.Stream()
    S.match_batch_dev(d, reads, offs, hits, stream=stream)
    S.locate_dev(d, hits, 4, 0, starts, pos, stream=stream)
    torch.mm(a, a, out=b)
    torch.cuda.synchronize()
    busy = torch.cuda.Event()
    with torch.cuda.stream(stream):
        for _ in range(60):  # about half a second
            torch.mm(a, a, out=b)
        busy.record()
    total = []
    locating = threading.Thread(target=lambda: total.append(S.locate_dev(d, hits, 4, 0, starts, pos, stream=stream)))
    locating.start()
    locating.join(0.05)
    assert locating.is_alive() and not busy.query()
    S.match_batch_dev(d, reads, offs, again, stream=stream)
    assert not busy.query(), "the batch was held back until the locate had returned"
    locating.join()
    torch.cuda.synchronize()
    assert total == [int(starts[-1])] and torch.equal(hits, again)


def test_host_locates_of_several_threads(index):
    """sa_locate of several threads at once, each with hits of its own."""
    _, sa, d = index
    wrong = []

    def work(seed):
        rng = np.random.default_rng(seed)
        for _ in range(20):
            count = int(rng.integers(1, 3000))
            lo = rng.integers(0, len(sa) - 40, count)
            rows = rng.integers(0, 40, count)
            hits = np.stack([lo, lo + rows, rows, np.ones(count, int)], 1).astype(np.int32)
            offs, pos = S.locate(d, hits, 16)
            take = np.minimum(rows, 16)
            want = [sa[a:a + t] for a, t in zip(lo, take)]
            if not (np.array_equal(np.diff(offs), take) and np.array_equal(pos, np.concatenate(want))):
                wrong.append(seed)

    threads = [threading.Thread(target=work, args=(k,)) for k in range(4)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not wrong
