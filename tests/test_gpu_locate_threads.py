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
