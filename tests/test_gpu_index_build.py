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
