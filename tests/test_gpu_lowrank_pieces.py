"""GPU parity of Q = X^T Phat, whose operands are cut into bf16 pieces: as good as fp32 products."""
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
    # the sum's roundings are at most one a row, the products left out and the pieces' rounding 3 * 2^-24 of a product
    tol = (rows + 8) * 2.0 ** -24
    for l, (m, n) in enumerate(shapes):
        o = int(batch.offsets[l])
        f = pay[offsets[l]:offsets[l] + 4 * (m + n) * rank].view(np.float32).astype(np.float64)
        p, got = f[:m * rank].reshape(m, rank), f[m * rank:].reshape(n, rank)
        x = batch.grads[o:o + m * n].reshape(m, n).astype(np.float64)
        assert (np.abs(got - x.T @ p) <= tol * (np.abs(x).T @ np.abs(p)) + 1e-300).all(), shapes[l]


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
