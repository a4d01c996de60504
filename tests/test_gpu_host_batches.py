"""Host batches on either side of the size up to which the search kernel reads
the pinned staging buffers itself, and of the reads a batch's chunks hold:
the same results as the device entry point gives."""
import numpy as np
import pytest

import paper_1303_3692_amd as S

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("count,length,kw", [(1, 0, {}), (1, 150, {}), (7, 1024, {}), (1000, 30, {}), (24_105, 150, {}),
                                             (24_106, 150, {}), (24_105, 150, dict(sort=1)), (24_105, 150, dict(defer=0)),
                                             (30_000, 150, {}), (4_003, 1024, {}), (1000, 30, dict(inline_pack=0))])
def test_host_batch_equals_device_batch(count, length, kw):
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    print("case: host batch", count, length, kw, flush=True)
    rng = np.random.default_rng(count)
    letters = np.frombuffer(b"ACGT", dtype=np.uint8)
    text = rng.choice(letters, 500_000)
    d = S.sa_build_device(text, 0)
    start = rng.integers(0, len(text) - 1024, count)
    data = text[start[:, None] + np.arange(length)].reshape(-1)
    if len(data):
        at = rng.integers(0, len(data), count // 2 + 1)
        data[at] = rng.choice(np.frombuffer(b"ACGTN", dtype=np.uint8), len(at))
    offs = np.arange(count + 1, dtype=np.int64) * length
    config = S.cfg(d, **kw)
    for _ in range(2):
        got = S.match_batch(d, data, offs, config=config)
        out = torch.full((count, 4), -7, dtype=torch.int32, device="cuda")
        d_data = torch.from_numpy(data if len(data) else np.zeros(1, np.uint8)).cuda()
        S.match_batch_dev(d, d_data, torch.from_numpy(offs).cuda(), out)
        torch.cuda.synchronize()
        assert (got == out.cpu().numpy()).all()
