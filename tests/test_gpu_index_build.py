"""Index construction on the device at the sizes where its kernels change
their ways: the packed and checked text around pieces and words, in both
cases and with a byte that is not a base at either end."""
import numpy as np
import pytest

import paper_1303_3692_amd as S

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module", autouse=True)
def device():
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")


@pytest.mark.parametrize("n", [1, 15, 16, 17, 31, 32, 33, 48, 63, 65, 4097])
def test_text_is_packed_and_checked(n, tmp_path):
    print("case: text of", n, flush=True)
    rng = np.random.default_rng(n)
    text = rng.choice(np.frombuffer(b"ACGTacgt", dtype=np.uint8), n)
    # the saved file holds the packed text and the suffix array
    S.sa_save(S.sa_build(text), str(tmp_path / "host"))
    S.sa_save(S.sa_download(S.sa_build_device(text, 0)), str(tmp_path / "device"))
    assert (tmp_path / "host").read_bytes() == (tmp_path / "device").read_bytes()
    for at in sorted({0, n // 2, n - 1}):
        for byte in (ord("N"), 0, ord("A") ^ 0x80, ord("@")):
            bad = text.copy()
            bad[at] = byte
            with pytest.raises(S.SaError) as e:
                S.sa_build_device(bad, 0)
            assert e.value.code == S.SA_EALPHABET and f"byte {at} " in str(e.value)


@pytest.mark.parametrize("kind", ["iid", "a", "tandem", "two letters"])
@pytest.mark.parametrize("k", [4, 5, 6, 7, 8, 11])
def test_prefix_table_entries(kind, k):
    """Every k-base string, as a read, gets from the table what a search from
    the root gives it, and so do the strings with two bases more: tables of
    one and of several workgroups, workgroups without rows and with all of
    them, and the suffixes shorter than k at the text's end."""
    print("case: table", kind, k, flush=True)
    n = 5_000
    rng = np.random.default_rng(k)
    text = {"iid": rng.integers(0, 4, n), "a": np.zeros(n, int), "tandem": np.tile(rng.integers(0, 4, 5), n // 5),
            "two letters": rng.integers(0, 2, n) * 3}[kind]
    d = S.sa_build_device(np.frombuffer(b"ACGT", dtype=np.uint8)[text], 0)
    d.set_prefix_table(k)
    for extra in (0, 2):
        m = k + extra
        count = 4 ** m
        v = torch.arange(count, device="cuda")
        if count > 1 << 20:
            v = torch.cat([v[:: count >> 18], v[-5000:], v[:5000]])
        digits = (v[:, None] >> (2 * torch.arange(m - 1, -1, -1, device="cuda"))) & 3
        reads = torch.tensor(list(b"ACGT"), dtype=torch.uint8, device="cuda")[digits].reshape(-1).contiguous()
        offs = torch.arange(len(v) + 1, device="cuda") * m
        outs = []
        for table in (1, 0):
            out = torch.full((len(v), 4), -7, dtype=torch.int32, device="cuda")
            S.match_batch_dev(d, reads, offs, out, config=S.cfg(d, prefix_table=table, sort=0))
            torch.cuda.synchronize()
            outs.append(out)
        assert torch.equal(*outs), (kind, k, extra)


def test_memory_of_a_freed_index_is_used_again_safely():
    """An index freed with a batch of it still running, the next one built at
    once (in the freed one's memory), also from several threads: every result
    is the one an index of its own gives."""
    import threading

    rng = np.random.default_rng(3)
    letters = np.frombuffer(b"ACGT", dtype=np.uint8)
    texts = [rng.choice(letters, 300_000) for _ in range(4)]
    count, m = 200_000, 60
    start = rng.integers(0, 300_000 - m, count)
    batches = []
    for t in texts:
        data = torch.from_numpy(t[start[:, None] + np.arange(m)].reshape(-1)).cuda()
        batches.append(data)
    offs = torch.arange(count + 1, device="cuda") * m
    keep = [S.sa_build_device(t, 0) for t in texts]
    want = []
    for d, data in zip(keep, batches):
        out = torch.zeros((count, 4), dtype=torch.int32, device="cuda")
        S.match_batch_dev(d, data, offs, out)
        torch.cuda.synchronize()
        want.append(out)
    del keep

    failures = []

    def work(which):
        stream = torch.cuda.Stream()
        for _ in range(3):
            for i in which:
                out = torch.full((count, 4), -7, dtype=torch.int32, device="cuda")
                torch.cuda.synchronize()
                d = S.sa_build_device(texts[i], 0)
                S.match_batch_dev(d, batches[i], offs, out, stream=stream)
                d.free()
                stream.synchronize()
                if not torch.equal(out, want[i]):
                    failures.append(i)

    work([0, 1, 2, 3])
    threads = [threading.Thread(target=work, args=([k, (k + 1) % 4],)) for k in range(4)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not failures
