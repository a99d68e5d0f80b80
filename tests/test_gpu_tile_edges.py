"""Kernels at the edges of their tiles: sizes of one tile, one more, one less, and ragged ends."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2607_01127_amd import logbq as L

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")]
DEV = "cuda:0"


@pytest.mark.parametrize("bits", [4, 8])
@pytest.mark.parametrize("n,k", [(1, 32), (31, 32), (32, 32), (33, 32), (9, 928), (2051, 4128)])
def test_dequantize_tiles(bits, n, k):
    """Tiles of 1024 weights per wavefront: below, at and above one, and more tiles than
    wavefronts; the buffer behind the result stays as it was. Looked-up values are exact."""
    print(f"dequantize bits={bits} n={n} k={k}", flush=True)
    rng = np.random.default_rng([bits, n, k])
    c = rng.integers(0, 1 << bits, size=(n, k), dtype=np.uint8)
    book = rng.standard_normal(1 << bits).astype(np.float32)
    packed = c if bits == 8 else c[:, 0::2] | (c[:, 1::2] << 4)
    out = torch.full((n * k + 64,), 7.0, device=DEV)
    call = L.dequantize if bits == 4 else L.dequantize8
    call(torch.from_numpy(packed).to(DEV), book, out=out[:n * k].view(n, k))
    got = out.cpu().numpy()
    assert np.array_equal(got[:n * k].reshape(n, k), book[c])
    assert np.all(got[n * k:] == 7.0)
