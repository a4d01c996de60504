"""Prefix tables whose strings have many rows each: the build searches the
rows of a workgroup instead of walking them."""
import time

import numpy as np
import pytest

import paper_1303_3692_amd as S

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

LETTERS = np.frombuffer(b"ACGT", dtype=np.uint8)


@pytest.fixture(scope="module", autouse=True)
def device():
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")


# 256 strings in a workgroup: 16 * 256 rows are walked, one more is searched.  A
# text of one letter has n - (k - 1) rows in the first workgroup of k bases.
WALKED = 16 * 256


@pytest.mark.parametrize("kind", ["iid", "a", "t", "tandem", "two letters", "ends short"])
@pytest.mark.parametrize("k,n", [(4, WALKED + 3), (4, WALKED + 4), (4, 300_000), (5, WALKED + 5), (6, 300_000), (7, 70_000)])
def test_entries_of_many_rows(kind, k, n):
    """Every k-base string, and with two bases more, as a read: what the table
    gives is what a search from the root gives."""
    print("case: table", kind, k, n, flush=True)
    rng = np.random.default_rng(k)
    text = {"iid": rng.integers(0, 4, n), "a": np.zeros(n, int), "t": np.full(n, 3),
            "tandem": np.resize(rng.integers(0, 4, 5), n), "two letters": rng.integers(0, 2, n) * 3,
            "ends short": np.concatenate([rng.integers(0, 4, n - 40), np.zeros(37, int), [1, 0, 0]])}[kind]
    d = S.sa_build_device(LETTERS[text], 0)
    d.set_prefix_table(k)
    for m in (k, k + 2):
        v = torch.arange(4 ** m, device="cuda")
        digits = (v[:, None] >> (2 * torch.arange(m - 1, -1, -1, device="cuda"))) & 3
        reads = torch.tensor(list(b"ACGT"), dtype=torch.uint8, device="cuda")[digits].reshape(-1).contiguous()
        offs = torch.arange(len(v) + 1, device="cuda") * m
        outs = []
        for table in (1, 0):
            out = torch.full((len(v), 4), -7, dtype=torch.int32, device="cuda")
            S.match_batch_dev(d, reads, offs, out, config=S.cfg(d, prefix_table=table, sort=0))
            torch.cuda.synchronize()
            outs.append(out)
        assert torch.equal(*outs), (kind, k, m)


def test_a_small_table_of_a_large_text_is_built_at_once():
    """4 M rows in a workgroup are not walked by it: 10 ms then, tens of
    microseconds searched."""
    n = 4_000_000
    rng = np.random.default_rng(0)
    for text in (rng.integers(0, 4, n), np.zeros(n, int)):
        d = S.sa_build_device(LETTERS[text], 0)
        took = []
        for _ in range(5):
            a = time.perf_counter()
            d.set_prefix_table(4)
            took.append(time.perf_counter() - a)
        print("case: table of 4 bases:", [round(1e6 * t) for t in took], "us", flush=True)
        assert min(took) < 2e-3
