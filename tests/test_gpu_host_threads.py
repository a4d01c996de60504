"""Host batches of several threads at once, on either side of the size up to
which the search kernel reads them in place."""
import threading

import numpy as np
import pytest

import paper_1303_3692_amd as S
from oracle import oracle

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

LETTERS = np.frombuffer(b"ACGT", dtype=np.uint8)


# one call reads 4 MiB in place (24,000 reads of 150 bases), two calls 1 MiB each
@pytest.mark.parametrize("nthreads,counts", [(1, (24_000, 24_200)), (2, (5_900, 6_200)), (4, (100, 2_900, 3_100)),
                                             (4, (1, 30_000))])
def test_batches_of_several_threads(nthreads, counts):
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    print("case: host batches", nthreads, counts, flush=True)
    rng = np.random.default_rng(nthreads)
    text = LETTERS[rng.integers(0, 4, 50_000)]
    d, sa = S.sa_build_device(text, 0), oracle.sa_build(text)
    batches = []
    for count in counts:
        start = rng.integers(0, len(text) - 150, count)
        data = text[start[:, None] + np.arange(150)].reshape(-1)
        change = rng.random(len(data)) < 0.005
        data[change] = LETTERS[rng.integers(0, 4, int(change.sum()))]
        offs = np.arange(count + 1, dtype=np.int64) * 150
        batches.append((data, offs, oracle.match(text, sa, data, offs)))
    wrong, ready = [], threading.Barrier(nthreads)

    def work(k):
        stream = torch.cuda.Stream()
        ready.wait()
        for i in range(12):
            data, offs, want = batches[(i + k) % len(batches)]
            got = S.match_batch(d, data, offs, stream=stream)
            if not ((got[:, :3] == want[:, :3]).all() and ((got[:, 3] & 1) == want[:, 3]).all()):
                wrong.append((k, i))

    threads = [threading.Thread(target=work, args=(k,)) for k in range(nthreads)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not wrong
