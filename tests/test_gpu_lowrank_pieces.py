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
