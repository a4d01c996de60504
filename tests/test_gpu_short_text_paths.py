"""Texts below 4096 bases: the paths that their settings lead to."""
import numpy as np
import pytest

import paper_1303_3692_amd as S
from oracle import oracle

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

LETTERS = np.frombuffer(b"ACGT", dtype=np.uint8)


@pytest.fixture(scope="module")
def index():
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    text = LETTERS[np.random.default_rng(5).integers(0, 4, 3_000)]
    return text, S.sa_build_device(text, 0)


def batch(text, count, lo, hi):
    """Reads of the text, one in twenty bases changed in every second one, some with an N."""
    rng = np.random.default_rng(count)
    m = rng.integers(lo, hi + 1, count)
    offs = np.zeros(count + 1, np.int64)
    np.cumsum(m, out=offs[1:])
    owner = np.repeat(np.arange(count), m)
    data = text[np.arange(offs[-1]) - offs[owner] + rng.integers(0, len(text) - hi, count)[owner]]
    change = (rng.random(len(data)) < 0.05) & (owner % 2 == 1)
    data[change] = LETTERS[rng.integers(0, 4, int(change.sum()))]
    data[(rng.random(len(data)) < 0.01) & (owner % 7 == 3)] = ord("N")
    return data, offs


@pytest.mark.parametrize("settings", [dict(sort=1, inline_pack=0), dict(sort=8, inline_pack=0), dict(sort=24, inline_pack=0),
                                      dict(sort=0, inline_pack=0), dict(sort=16), dict(sort=0, prefix_table=0), {}],
                         ids=str)
@pytest.mark.parametrize("count", [1, 65, 5_000])
def test_settings(index, settings, count):
    """The packed and sorted paths, which a short text takes only without
    inline packing, and the others give the oracle's results."""
    text, d = index
    print("case: short text", settings, count, flush=True)
    data, offs = batch(text, count, 1, 700)
    out = torch.full((count, 4), -7, dtype=torch.int32, device="cuda")
    S.match_batch_dev(d, torch.from_numpy(data).cuda(), torch.from_numpy(offs).cuda(), out, config=S.cfg(d, **settings))
    torch.cuda.synchronize()
    got, want = out.cpu().numpy(), oracle.match(text, oracle.sa_build(text), data, offs)
    assert (got[:, :3] == want[:, :3]).all() and ((got[:, 3] & 1) == want[:, 3]).all()


def test_noalloc_takes_what_needs_no_packed_arrays(index):
    """A batch beyond the fixed scratch's packed reads, with the settings that
    such a text has by default: it is searched without packed arrays."""
    text, d = index
    count = S.sa_noalloc_max_reads(True) + 1
    print("case: noalloc, short text,", count, "reads", flush=True)
    data, offs = batch(text, count, 1, 12)
    reads, starts = torch.from_numpy(data).cuda(), torch.from_numpy(offs).cuda()
    outs = []
    for call in (S.match_batch_dev, S.match_batch_dev_noalloc):
        out = torch.full((count, 4), -7, dtype=torch.int32, device="cuda")
        call(d, reads, starts, out)
        torch.cuda.synchronize()
        outs.append(out)
    assert torch.equal(*outs)
    with pytest.raises(S.SaError) as e:
        S.match_batch_dev_noalloc(d, reads, starts, outs[0], config=S.cfg(d, inline_pack=0))
    assert e.value.code == S.SA_ENOSPC
