"""Memory of a freed index while another stream is being captured."""
import time

import numpy as np
import pytest

import paper_1303_3692_amd as S

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module", autouse=True)
def device():
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")


def test_capture_while_kept_memory_is_given_back():
    """An index is freed just before a capture in global mode, which stays
    open until the index's memory has been given back (after 2 s): the
    capture ends cleanly, and its graph replays right."""
    text = np.random.default_rng(1).choice(np.frombuffer(b"ACGT", dtype=np.uint8), 1_000_000)
    x = torch.zeros(1000, device="cuda")
    y = torch.empty_like(x)
    torch.add(x, 1, out=y)
    index = S.sa_build_device(text, 0)
    torch.cuda.synchronize()
    before = torch.cuda.mem_get_info()[0]
    index.free()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, capture_error_mode="global"):
        torch.add(x, 1, out=y)
        time.sleep(3)
    for i in range(3):
        x.fill_(i)
        graph.replay()
        torch.cuda.synchronize()
        assert (y == i + 1).all()
    # the table alone took 4^12 entries of 16 bytes
    assert torch.cuda.mem_get_info()[0] - before >= 16 << 24


def test_trim():
    """Kept memory is given back at once when that is asked for."""
    text = np.random.default_rng(1).choice(np.frombuffer(b"ACGT", dtype=np.uint8), 1_000_000)
    S.sa_trim()
    index = S.sa_build_device(text, 0)
    size = sum(index.index_bytes().values())
    torch.cuda.synchronize()
    before = torch.cuda.mem_get_info()[0]
    index.free()
    given = S.sa_trim()
    assert size <= given <= size + 8 * 256 and S.sa_trim() == 0
    assert torch.cuda.mem_get_info()[0] - before >= 16 << 24
    with pytest.raises(S.SaError) as e:
        S.sa_trim(-1)
    assert e.value.code == S.SA_EINVAL
