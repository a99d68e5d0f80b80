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


def _gptq_case(n, k, seed):
    rng = np.random.default_rng(seed)
    w = (0.02 * rng.standard_t(4, size=(n, k))).astype(np.float32)
    u = np.triu(0.1 * rng.standard_normal((k, k)), 1).astype(np.float32)
    u[np.arange(k), np.arange(k)] = np.exp(rng.normal(0, 0.5, k)).astype(np.float32)
    return rng, w, u


def _special_rows(rng, w, u):
    """Values whose errors the short division does not cover: zeros of both signs, subnormal, tiny
    and huge weights, infinities and NaN, and extreme diagonal entries of U."""
    n, k = w.shape
    w[:, 5] = 0.0
    w[:, 6] = -0.0
    w[0, ::3] = 0.0
    w[1 % n, ::3] = -0.0
    w[2 % n] *= np.float32(1e-36)
    w[3 % n] *= np.float32(1e30)
    w[4 % n, 17 % k] = np.inf
    w[5 % n, k - 1] = -np.inf
    w[6 % n, 3] = np.nan
    u[7, 7] = np.float32(1e-30)
    if k > 200:
        u[150, 150] = np.float32(1e25)
        u[40, 45:] = 0.0
        u[41, 50:] = -0.0


@pytest.mark.parametrize("n,k", [(1, 32), (15, 64), (17, 96), (16, 128), (65, 224), (33, 256)])
@pytest.mark.parametrize("book", ["mirrored", "any", "uniform"])
@pytest.mark.parametrize("special", [False, True])
def test_gptq_edges(n, k, book, special):
    """Ragged rows and last blocks, and values outside the short division's range, for each kind of
    codebook, bit for bit against the CPU oracle's float32 loop."""
    from oracle import gptq_oracle as G
    print(f"gptq edges n={n} k={k} {book} special={special}", flush=True)
    rng, w, u = _gptq_case(n, k, [7, n, k])
    fit_on = (0.02 * rng.standard_t(4, size=4096)).astype(np.float32)
    p = L.fit_uniform(fit_on) if book == "uniform" else L.fit(fit_on)
    if book == "any":
        for i in range(1, 8):
            p.codebook[8 + i] *= 1.125
        p.codebook[0] = 0.001
    if special:
        _special_rows(rng, w, u)
    levels, th = p.codebook_array(), np.ctypeslib.as_array(p.thresholds).copy()

    def quantize(col):
        if book == "uniform":
            c = np.sum(col[:, None] >= th[None, :15], axis=1)
        else:
            c = np.sum(np.abs(col)[:, None] >= th[None, :7], axis=1)
            c = np.where((col < 0) & (c > 0), c + 8, c)
        return c.astype(np.uint8), levels[c]

    with np.errstate(all="ignore"):
        codes_ref, w_ref = G.gptq(w, u, quantize)
    wd = torch.from_numpy(w.copy()).to(DEV)
    codes = L.gptq(wd, torch.from_numpy(u).to(DEV), p)
    got, wg = codes.cpu().numpy(), wd.cpu().numpy()
    assert np.array_equal(got, codes_ref[:, 0::2] | (codes_ref[:, 1::2] << 4))
    same = (wg.view(np.uint32) == w_ref.view(np.uint32)) | (np.isnan(wg) & np.isnan(w_ref))
    assert same.all(), f"{np.count_nonzero(~same)} of {same.size} weights differ"


def _gptq_book(book, rng):
    """Parameters of a codebook of each kind, and its quantizer for the oracle."""
    fit_on = (0.02 * rng.standard_t(4, size=4096)).astype(np.float32)
    p = L.fit_uniform(fit_on) if book == "uniform" else L.fit(fit_on)
    if book == "any":
        for i in range(1, 8):
            p.codebook[8 + i] *= 1.125
        p.codebook[0] = 0.001
    levels, th = p.codebook_array(), np.ctypeslib.as_array(p.thresholds).copy()

    def quantize(col):
        if book == "uniform":
            c = np.sum(col[:, None] >= th[None, :15], axis=1)
        else:
            c = np.sum(np.abs(col)[:, None] >= th[None, :7], axis=1)
            c = np.where((col < 0) & (c > 0), c + 8, c)
        return c.astype(np.uint8), levels[c]
    return p, levels, quantize


@pytest.mark.parametrize("book", ["mirrored", "any", "uniform"])
@pytest.mark.parametrize("col", [0, 5, 37, 150])
def test_gptq_minus_zero(book, col):
    """A weight of -0 that no earlier error has moved is -0 when its column is quantized and is
    returned as -0, whatever the errors of later columns; every other value is ordinary, so no
    row takes the general form for another reason. Weights and the last block's errors bit for
    bit against the CPU oracle's float32 loop."""
    from oracle import gptq_oracle as G
    n, k = 40, 160
    print(f"gptq -0 {book} column {col}", flush=True)
    rng, w, u = _gptq_case(n, k, [11, col])
    p, levels, quantize = _gptq_book(book, rng)
    # Every other row starts with values of the codebook, whose errors are +0, and keeps its -0;
    # in the others a negative error times the zeros of U turns it to +0 (column 0: in none).
    w[::2, :col] = levels[rng.integers(1, 8, (n // 2, col))]
    w[:, col] = -0.0
    u[:col, col] = 0.0
    codes_ref, w_ref = G.gptq(w, u, quantize)
    assert not w_ref[:, col].any() and np.signbit(w_ref[::2, col]).all()
    wd = torch.from_numpy(w.copy()).to(DEV)
    err = torch.full((n, L.GPTQ_BLOCK), float("nan"), device=DEV)
    codes = L.gptq(wd, torch.from_numpy(u).to(DEV), p, workspace=err)
    assert np.array_equal(codes.cpu().numpy(), codes_ref[:, 0::2] | (codes_ref[:, 1::2] << 4))
    wrong = wd.cpu().numpy().view(np.uint32) != w_ref.view(np.uint32)
    assert not wrong.any(), f"{np.count_nonzero(wrong)} weights differ"
    last = (w_ref[:, 128:] - levels[codes_ref[:, 128:]]) / np.diag(u)[128:]
    wrong = err[:, :32].cpu().numpy().view(np.uint32) != last.view(np.uint32)
    assert not wrong.any(), f"{np.count_nonzero(wrong)} errors differ"


@pytest.mark.parametrize("bits", [4, 8])
@pytest.mark.parametrize("n,k,m", [(16640, 32, 257), (16385, 96, 320), (16383, 544, 513),
                                   (4097, 1056, 2049), (14336, 64, 1024), (4096, 14336, 1025),
                                   (16641, 224, 193), (20001, 1056, 129), (1025, 8160, 1300)])
def test_prefill_tiles(bits, n, k, m):
    """Prefill tiles of 256 weight rows x 64 to 256 batch rows and steps of 64 k: one row past a
    tile, one short of it, part steps, one and two K parts; a fitted-like and an arbitrary codebook
    against float64, y prefilled with NaN, the buffer behind it as it was, two calls bit-equal. The
    bound is the rounding of a codebook entry to float16, 2^-11, plus k float32 sums."""
    assert L.linear_path(bits, m, k, n) == "mfma_pf"
    print(f"prefill bits={bits} n={n} k={k} m={m} {L.linear_kernel(bits, m, k, n)}", flush=True)
    rng = np.random.default_rng([bits, n, k, m])
    c = torch.from_numpy(rng.integers(0, 256, size=(n, k * bits // 8), dtype=np.uint8)).to(DEV)
    x = torch.from_numpy(rng.standard_normal((m, k)).astype(np.float16)).to(DEV)
    half = (1 << (bits - 1)) - 1
    mag = np.concatenate([[0], 1.5 ** (np.linspace(-6, 0, half))])
    pick = rng.choice(m, 40, replace=False)
    pick[:2] = 0, m - 1
    for book in (np.concatenate([mag, -mag]), rng.standard_normal(1 << bits)):
        book = book.astype(np.float32)
        buf = torch.full((m * n + 64,), float("nan"), device=DEV)
        buf[m * n:] = 7.0
        y = buf[:m * n].view(m, n)
        call = L.linear if bits == 4 else L.linear8
        call(x, c, book, out=y)
        y2 = call(x, c, book)
        assert torch.equal(y, y2) and bool((buf[m * n:] == 7.0).all())
        table = torch.tensor(book.astype(np.float64), device=DEV)
        w = table[c.int()] if bits == 8 else torch.stack(
            [table[(c & 15).int()], table[(c >> 4).int()]], dim=2).reshape(n, k)
        xs = x[torch.from_numpy(pick).to(DEV)].double()
        bound = (xs.abs() @ w.abs().T.contiguous()) * (2.0 ** -11 + k * 2.0 ** -24)
        got = y[torch.from_numpy(pick).to(DEV)].double()
        assert bool(((got - xs @ w.T.contiguous()).abs() <= bound).all())


@pytest.mark.parametrize("n,k", [(130, 512), (33, 1056), (40, 4128), (4097, 4064), (2047, 8160),
                                 (2049, 8224), (1025, 11008), (4099, 16352), (16399, 2080),
                                 (32785, 2080)])
def test_ragged_split_k(n, k):
    """Split-K at K outside its powers of two: a last wavefront with one column block of 32 or all
    but one, one and two K parts, a partial last block of rows. Single calls repeat their bits, a
    grouped call equals them, and another codebook (which takes another kernel) agrees too, all
    within the float16 rounding of the codebook, 2^-11, plus k float32 sums."""
    rng = np.random.default_rng([n, k])
    c = torch.from_numpy(rng.integers(0, 256, size=(n, k // 2), dtype=np.uint8)).to(DEV)
    mag = np.concatenate([[0], 1.5 ** np.linspace(-6, 0, 7)])
    books = [np.concatenate([mag, -mag]).astype(np.float32),
             rng.standard_normal(16).astype(np.float32)]
    for m in (3, 4, 6, 8, 9, 16):
        print(f"ragged split-K n={n} k={k} m={m} {L.linear_kernel(4, m, k, n)}", flush=True)
        x = torch.from_numpy(rng.standard_normal((m, k)).astype(np.float16)).to(DEV)
        ys = []
        for book in books:
            y = torch.full((m, n), float("nan"), device=DEV)
            L.linear(x, c, book, out=y)
            assert torch.equal(y, L.linear(x, c, book))
            table = torch.tensor(book.astype(np.float64), device=DEV)
            w = torch.stack([table[(c & 15).int()], table[(c >> 4).int()]], dim=2).reshape(n, k)
            bound = (x.double().abs() @ w.abs().T.contiguous()) * (2.0 ** -11 + k * 2.0 ** -24)
            assert bool(((y.double() - x.double() @ w.T.contiguous()).abs() <= bound).all())
            ys.append(y)
        for a, b in zip(L.linear_multi(x, [c, c], books), ys):
            assert torch.equal(a, b)
        for a, b in zip(L.linear_multi(x, [c, c[:16]], [books[0]] * 2), (ys[0], None)):
            if b is not None:
                assert torch.equal(a, b)
            else:
                assert torch.equal(a, L.linear(x, c[:16], books[0]))


@pytest.mark.parametrize("n,k", [(130, 512), (33, 1056), (2047, 2080), (2049, 4128), (4097, 6112),
                                 (2048, 6176), (4096, 8160), (16399, 1056), (32785, 2080)])
def test_ragged_split_k8(n, k):
    """8-bit split-K at K outside its powers of two: one to four phases per wavefront, a last one
    with 32 columns or all but 32, wavefronts with none, a partial last block of rows; two calls
    bit-equal, within the float16 rounding of the codebook, 2^-11, plus k float32 sums."""
    rng = np.random.default_rng([8, n, k])
    c = torch.from_numpy(rng.integers(0, 256, size=(n, k), dtype=np.uint8)).to(DEV)
    book = rng.standard_normal(256).astype(np.float32)
    w = torch.tensor(book.astype(np.float64), device=DEV)[c.int()]
    for m in (3, 4, 6, 8, 9, 12, 16):
        print(f"ragged split-K 8 n={n} k={k} m={m} {L.linear_kernel(8, m, k, n)}", flush=True)
        x = torch.from_numpy(rng.standard_normal((m, k)).astype(np.float16)).to(DEV)
        y = torch.full((m, n), float("nan"), device=DEV)
        L.linear8(x, c, book, out=y)
        assert torch.equal(y, L.linear8(x, c, book))
        bound = (x.double().abs() @ w.abs().T.contiguous()) * (2.0 ** -11 + k * 2.0 ** -24)
        assert bool(((y.double() - x.double() @ w.T.contiguous()).abs() <= bound).all())
