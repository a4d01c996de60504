"""Locate at the sizes where its kernels change their ways: reads around a
workgroup and a tile, more rounds per tile, and so many tiles that a kernel of
its own adds up their sums.  The hits are made up (any interval inside the
text will do); positions and offsets are checked against the suffix array."""
import numpy as np
import pytest

import paper_1303_3692_amd as S

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("nreads,cap", [(1, 3), (255, 1), (256, 300), (257, 300), (1025, 4), (262_144, 5), (600_001, 2),
                                        (8_400_000, 3)])
def test_offsets_and_positions(nreads, cap):
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    print("case: locate", nreads, cap, flush=True)
    n = 20_000
    text = np.random.default_rng(1).choice(np.frombuffer(b"ACGT", dtype=np.uint8), n)
    host = S.sa_build(text)
    d = S.sa_upload(host, 0)
    sa = torch.from_numpy(host.suffix_array()).cuda()
    i = torch.arange(nreads, device="cuda")
    lo = (i * 7919) % (n - 400)
    rows = torch.where(i % 11 == 0, i % 400, i % 3)  # long lists among short and empty ones
    flags = (i % 5 != 2).long()
    hits = torch.stack([lo, lo + rows, i % 50, flags], 1).int()
    count = torch.where(flags == 1, rows.clamp(max=cap), 0)
    want = torch.zeros(nreads + 1, dtype=torch.int64, device="cuda")
    want[1:] = torch.cumsum(count, 0)
    total = int(want[-1])
    owner = torch.repeat_interleave(i, count)
    positions = sa[lo[owner] + torch.arange(total, device="cuda") - want[owner]]
    for room in (total, total - 1):  # the whole list, and one position too many
        offs = torch.full((nreads + 1,), -7, dtype=torch.int64, device="cuda")
        pos = torch.full((max(room, 1) + 3,), -7, dtype=torch.int32, device="cuda")
        if room == total:
            assert S.locate_dev(d, hits, cap, 0, offs, pos[:room]) == total
            torch.cuda.synchronize()
            assert torch.equal(pos[:total], positions)
        elif room >= 0:
            with pytest.raises(S.SaError) as e:
                S.locate_dev(d, hits, cap, 0, offs, pos[:room])
            assert e.value.code == S.SA_ENOSPC
            torch.cuda.synchronize()
            assert bool((pos == -7).all())
        else:
            continue
        assert torch.equal(offs, want) and bool((pos[max(room, 0):] == -7).all())


@pytest.mark.parametrize("nreads", [3, 70_000, 3_000_000])
def test_offsets_are_whole_when_the_call_returns(nreads):
    """Another stream that does not wait for the call's, and the host form,
    see every offset once the call has returned."""
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    print("case: locate offsets at return", nreads, flush=True)
    n = 20_000
    text = np.random.default_rng(1).choice(np.frombuffer(b"ACGT", dtype=np.uint8), n)
    d = S.sa_upload(S.sa_build(text), 0)
    i = torch.arange(nreads, device="cuda")
    lo = (i * 7919) % (n - 400)
    rows = i % 4
    hits = torch.stack([lo, lo + rows, i % 50, torch.ones_like(i)], 1).int()
    want = torch.zeros(nreads + 1, dtype=torch.int64, device="cuda")
    want[1:] = torch.cumsum(rows, 0)
    total = int(want[-1])
    pos = torch.empty(total, dtype=torch.int32, device="cuda")
    side = torch.cuda.Stream()
    torch.cuda.synchronize()
    for _ in range(5):
        offs = torch.full((nreads + 1,), -7, dtype=torch.int64, device="cuda")
        torch.cuda.synchronize()
        assert S.locate_dev(d, hits, 4, 0, offs, pos) == total
        with torch.cuda.stream(side):
            seen = offs.clone()
        torch.cuda.synchronize()
        assert torch.equal(seen, want)
    host_offs, host_pos = S.locate(d, hits.cpu().numpy(), 4, 0)
    assert np.array_equal(np.asarray(host_offs), want.cpu().numpy()) and len(host_pos) == total
