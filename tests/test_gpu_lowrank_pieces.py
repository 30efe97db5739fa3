"""GPU parity of P = X Q0 and Q = X^T Phat, whose operands are cut into bf16 pieces: as good as fp32 products."""
import numpy as np
import pytest

from paper_2210_17357_amd import workloads as W

from gpu_util import tables, to_device, torch_cuda

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("scale", (1e-12, 1.0, 1e12))
@pytest.mark.parametrize("rows", (1, 31, 32, 33, 64, 97, 200))
def test_second_contraction_is_an_fp32_product(rows, scale):
    from paper_2210_17357_amd import binding as B
    torch = torch_cuda()
    rank = min(rows, 8)
    rng = np.random.default_rng(rows)
    shapes = ((rows, 5), (rows, 127), (rows, 128), (rows, 129), (rows, 161))
    w = W.Workload("pieces", shapes, ((W.LOWRANK, float(rank)),), 0, 100, "lowrank64", "normal0.1", (-3.0, -1.0), r_max=64)
    batch = W.generate(w)
    # magnitudes over eight decades beside each other, every bit of the significand in use
    batch.grads[:] = (rng.standard_normal(batch.grads.size) * 10.0 ** rng.uniform(-4, 4, batch.grads.size) * scale).astype(np.float32)
    batch.ef[:] = 0
    L = len(shapes)
    choice = np.zeros(L, np.int32)
    layers, ctab = tables(batch, list(w.candidates))
    g, e, q = to_device(batch)
    h = B.Handle(int(batch.grads.size), L, 1, r_max=64)
    offsets = B.payload_layout(layers, ctab, choice)
    payload = torch.zeros(int(offsets[-1]) + 16, dtype=torch.uint8, device="cuda")
    h.compress(g, e, layers, ctab, choice, payload, offsets, q)
    pay = payload.cpu().numpy()
    h.close()
    # the sum's roundings are at most one a row, eight for the products of a row's pieces
    tol = (rows + 8) * 2.0 ** -24
    for l, (m, n) in enumerate(shapes):
        o = int(batch.offsets[l])
        f = pay[offsets[l]:offsets[l] + 4 * (m + n) * rank].view(np.float32).astype(np.float64)
        p, got = f[:m * rank].reshape(m, rank), f[m * rank:].reshape(n, rank)
        x = batch.grads[o:o + m * n].reshape(m, n).astype(np.float64)
        assert (np.abs(got - x.T @ p) <= tol * (np.abs(x).T @ np.abs(p)) + 1e-300).all(), shapes[l]


# One product, formed as eight on the matrix unit: the largest, exact, and seven whose sum is at most 2^-6 of it, each
# addition of which is within 2^-23 of what it gives; their sum is rounded once more.
PRODUCT = 2.0 ** -24 + 7 * 2.0 ** -6 * 2.0 ** -23 + 2.0 ** -32


def _factors(x, q0, rank, one_call=False):
    """Phat and Q of one matrix, compressed from a zero error feedback; one_call: without one, where the first contraction is
    another kernel."""
    from paper_2210_17357_amd import binding as B
    torch = torch_cuda()
    m, n = x.shape
    layers, ctab = B.layer_table([0], [m * n], [m], [n]), B.cand_table([(W.LOWRANK, float(rank))])
    choice = np.zeros(1, np.int32)
    g = torch.from_numpy(np.ascontiguousarray(x, np.float32).ravel()).cuda()
    q = torch.from_numpy(np.ascontiguousarray(q0, np.float32).ravel()).cuda()
    h = B.Handle(m * n, 1, 1, r_max=q0.shape[1])
    offsets = B.payload_layout(layers, ctab, choice)
    payload = torch.zeros(int(offsets[-1]) + 16, dtype=torch.uint8, device="cuda")
    if one_call:
        h.set_ef_zero_on_entry(True)
        h.profile_solve_compress(g, torch.zeros_like(g), layers, ctab, 0, 10, payload, q)
    else:
        h.compress(g, torch.zeros_like(g), layers, ctab, choice, payload, offsets, q)
    f = payload.cpu().numpy()[:4 * (m + n) * rank].view(np.float32).astype(np.float64)
    h.close()
    return f[:m * rank].reshape(m, rank), f[m * rank:].reshape(n, rank)


def _values(kind, rng, n):
    if kind == "random":
        return (rng.uniform(1, 2, n) * rng.choice((-1, 1), n)).astype(np.float32)
    # the second piece as large as it can be and the third half a step of it, with one sign in every product
    v = np.array([0x3F80FF80], np.uint32).view(np.float32)[0]
    return (v * 2.0 ** rng.integers(-3, 4, n)).astype(np.float32)


# X and Q0 so small that their third pieces are below what bf16 holds (from 2^-110 down), or not
SCALES = ((1.0, 1.0), (2.0 ** -116, 1.0), (1.0, 2.0 ** -116), (2.0 ** -109, 1.0), (2.0 ** -64, 2.0 ** -52))


@pytest.mark.parametrize("scale_x,scale_q", SCALES)
@pytest.mark.parametrize("kind", ("random", "worst"))
def test_single_products_of_the_first_contraction(kind, scale_x, scale_q):
    """Rows with one value: each row of P is one product.  Phat is P times a factor that rows whose product is exact tell."""
    rng = np.random.default_rng(5)
    m, n, exact = 65500, 600, 4096                          # a last tile of few rows, two ranges of columns
    col = rng.integers(1, n, m)
    col[:exact] = 0
    value = _values(kind, rng, m)
    value[:exact] = rng.uniform(1, 2, exact)
    value *= np.float32(scale_x)
    x, q0 = np.zeros((m, n), np.float32), _values(kind, rng, n)[:, None] * np.float32(scale_q)
    x[np.arange(m), col] = value
    q0[0] = scale_q
    phat = _factors(x, q0, 1)[0][:, 0]
    want = value.astype(np.float64) * q0[col, 0]
    half = np.spacing(np.abs(phat).astype(np.float32)).astype(np.float64) / 2
    low = ((np.abs(phat) - half) / np.abs(want))[:exact].max()
    high = ((np.abs(phat) + half) / np.abs(want))[:exact].min()
    assert low <= high * (1 + 1e-12) and high / low - 1 < 2.0 ** -30
    assert (np.abs(phat / (want * (low + high) / 2) - 1) <= PRODUCT + 2.0 ** -24 + 2.0 ** -30).all()


@pytest.mark.parametrize("scale", (1.0, 2.0 ** -116, 2.0 ** -109))
@pytest.mark.parametrize("kind", ("random", "worst"))
def test_single_products_of_the_second_contraction(kind, scale):
    """Columns with one value: each row of Q is one product of it with a row of Phat."""
    rng = np.random.default_rng(6)
    m, n = 67, 32700
    row = rng.integers(0, m, n)
    value = _values(kind, rng, n) * np.float32(scale)
    x = np.zeros((m, n), np.float32)
    x[row, np.arange(n)] = value
    phat, q = _factors(x, rng.standard_normal((n, 64)), 8)
    want = value.astype(np.float64)[:, None] * phat[row]
    assert (np.abs(q - want) <= PRODUCT * np.abs(want) + 2.0 ** -149).all()


@pytest.mark.parametrize("scale", (2.0 ** -100, 2.0 ** -116, 2.0 ** -122))
def test_small_matrices_in_the_one_call(scale):
    """Without an error feedback the first contraction is another kernel."""
    from paper_2210_17357_amd import binding as B
    torch = torch_cuda()
    rng = np.random.default_rng(7)
    m, n, rank = 150, 700, 4
    x = (rng.standard_normal((m, n)) * scale).astype(np.float32)
    q0 = rng.standard_normal((n, 64)).astype(np.float32)
    layers, ctab = B.layer_table([0], [m * n], [m], [n]), B.cand_table([(W.LOWRANK, float(rank))])
    h = B.Handle(m * n, 1, 1, r_max=64)
    h.set_ef_zero_on_entry(True)
    payload = torch.zeros(4 * (m + n) * rank + 32, dtype=torch.uint8, device="cuda")
    g, q = torch.from_numpy(x.ravel()).cuda(), torch.from_numpy(q0.ravel()).cuda()
    h.profile_solve_compress(g, torch.zeros_like(g), layers, ctab, 0, 10, payload, q)
    f = payload.cpu().numpy()[:4 * (m + n) * rank].view(np.float32).astype(np.float64)
    h.close()
    x64 = x.astype(np.float64) / scale
    ortho, r = np.linalg.qr(x64 @ q0.astype(np.float64))
    phat = (ortho * np.sign(np.diag(r)))[:, :rank]
    got = f[:m * rank].reshape(m, rank)
    # sums of 700 fp32 products, and a condition number below 4 of the leading columns
    assert np.linalg.norm(got - phat) <= 4 * 30 * 2.0 ** -24 * np.linalg.norm(phat)
    want = x64.T @ got
    assert np.linalg.norm(f[m * rank:].reshape(n, rank) / scale - want) <= 150 * 2.0 ** -24 * np.linalg.norm(want) + 2.0 ** -149 / scale * n


@pytest.mark.parametrize("one_call", (False, True))
@pytest.mark.parametrize("small", ("x", "q0"))
@pytest.mark.parametrize("m,n", ((3, 3), (33, 65), (97, 600), (700, 130)))
def test_smallest_values_are_not_zero(m, n, small, one_call):
    """X, or Q0, of whole multiples of the smallest fp32 value, all too small for any piece; products and sums of P are exact."""
    rng = np.random.default_rng(8)
    x = rng.integers(-1000, 1000, (m, n)) * (rng.random((m, n)) < 0.02)
    x[m // 2, n // 2] = 999
    q0 = rng.choice((-2, -1, 1, 2), (n, 1))
    least = 2.0 ** -149
    phat, q = _factors(x * least, q0, 1, one_call) if small == "x" else _factors(x, q0 * least, 1, one_call)
    p = (x @ q0).astype(np.float64)
    assert np.linalg.norm(phat - p / np.linalg.norm(p)) <= 2.0 ** -21
    # each product of Q and each addition is rounded once, to the smallest value where X is
    unit = least if small == "x" else 1.0
    assert (np.abs(q / unit - x.T @ phat) <= 2 * m * (1.0 if small == "x" else 2.0 ** -23 * (np.abs(x).T @ np.abs(phat)))).all()


def test_zero_matrices_stay_zero():
    x, q0 = np.zeros((70, 300), np.float32), np.random.default_rng(9).standard_normal((300, 8))
    for factor in _factors(x, q0, 4) + _factors(x + 1.0, np.zeros_like(q0), 4) + _factors(x, q0, 4, one_call=True):
        assert not factor.any()


@pytest.mark.parametrize("rank", (2, 3, 4, 5, 15, 16, 17, 24, 32, 34))
def test_reconstruction_at_groups_of_ranks_and_tiles(rank):
    """Ranks around the groups that are loaded and multiplied together, matrices around the tiles of 32 x 32 and the
    128 columns of a workgroup, on whole lines and off them, payload rows shorter than a load."""
    from test_gpu_decompress import _roundtrip
    shapes = ((32, 128), (31, 127), (33, 129), (64, 160), (1, 32), (65, 97), (32, 1), (96, 288), (34, 34), (128, 64))
    w = W.Workload("groups", shapes, ((W.LOWRANK, float(rank)),), 0, 100, "lowrank64", "normal0.1", (-3.0, -1.0), r_max=64)
    batch = W.generate(w)
    # the image is a product of `rank` fp32 terms an element; in the norm at most rank * 2^-24 * sqrt(rank) relative
    # to the image of orthonormal columns, well inside this
    _roundtrip(w, batch, np.zeros(len(shapes), np.int32), fro_tol=1e-5)


@pytest.mark.parametrize("rank", (3, 16, 17, 40))
def test_feedback_is_what_the_payload_leaves(rank):
    from paper_2210_17357_amd import binding as B
    torch = torch_cuda()
    shapes = ((32, 128), (31, 127), (33, 129), (64, 160), (200, 33), (65, 97), (96, 288), (128, 64))
    cands = ((W.LOWRANK, float(rank)), (W.LOWRANK, 64.0))
    w = W.Workload("left", shapes, cands, 0, 100, "lowrank64", "normal0.1", (-3.0, -1.0), r_max=64)
    batch = W.generate(w)
    L = len(shapes)
    layers, ctab = tables(batch, list(cands))
    g, e, q = to_device(batch)
    h = B.Handle(int(batch.grads.size), L, 2, r_max=64)
    capacity = int(B.sizes(layers, ctab, 128).max(axis=1).sum()) + 16 * (L + 1)
    payload = torch.zeros(capacity // 16 * 16 + 16, dtype=torch.uint8, device="cuda")
    # the one call: factors out of the profile's scratch, every layer at the default (E_max is its error, few bins)
    out = h.profile_solve_compress(g, e, layers, ctab, 0, 1, payload, q)
    choice = out[4]
    offsets = B.payload_layout(layers, ctab, choice)
    pay, left = payload.cpu().numpy(), e.cpu().numpy()
    h.close()
    for l, (m, n) in enumerate(shapes):
        r = int(cands[choice[l]][1])
        o = int(batch.offsets[l])
        f = pay[offsets[l]:offsets[l] + 4 * (m + n) * r].view(np.float32).astype(np.float64)
        image = f[:m * r].reshape(m, r) @ f[m * r:].reshape(n, r).T
        x = (batch.grads[o:o + m * n] + batch.ef[o:o + m * n]).astype(np.float64)
        tol = (r + 2) * 2.0 ** -24 * (r ** 0.5 + 1.0)        # as for every sum of r + 1 terms, see the receiver's test
        assert np.linalg.norm(left[o:o + m * n] - (x - image.ravel())) <= tol * np.linalg.norm(x), (l, r)
