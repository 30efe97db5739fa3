"""GPU parity, receiver side: lgreco_decompress against the oracle's decompress_layer on the
payloads the GPU sender wrote (which are themselves checked against the oracle's payloads)."""
import numpy as np
import pytest

from oracle import pipeline
from paper_2210_17357_amd import workloads as W

from gpu_util import tables, to_device, torch_cuda

pytestmark = pytest.mark.gpu


def _roundtrip(w, batch, choice, stochastic=False, fro_tol=None):
    from paper_2210_17357_amd import binding as B
    torch = torch_cuda()
    cands = list(w.candidates)
    layers, ctab = tables(batch, cands)
    g, e, q = to_device(batch)
    if e is None:
        e = torch.zeros_like(g)
    L = len(batch.numels)
    h = B.Handle(int(batch.grads.size), L, len(cands), stochastic=stochastic, seed=w.seed, r_max=w.r_max)
    offsets = B.payload_layout(layers, ctab, choice)
    payload = torch.zeros(int(offsets[-1]) + 16, dtype=torch.uint8, device="cuda")
    h.compress(g, e.clone(), layers, ctab, choice, payload, offsets, None if q is None else q.clone())
    pay = payload.cpu().numpy()
    total = int(batch.grads.size)
    sentinel = np.float32(123.5)
    out = torch.full((total,), float(sentinel), dtype=torch.float32, device="cuda")
    h.decompress(payload, offsets, layers, ctab, choice, out, accumulate=False)
    got = out.cpu().numpy()
    base = (np.arange(total) % 17).astype(np.float32) * np.float32(1e-3)
    acc = torch.from_numpy(base).cuda()
    h.decompress(payload, offsets, layers, ctab, choice, acc, accumulate=True)
    got_acc = acc.cpu().numpy()
    covered = np.zeros(total, bool)
    for l in range(L):
        off, n = int(batch.offsets[l]), int(batch.numels[l])
        covered[off:off + n] = True
        cand = cands[choice[l]]
        size = int(offsets[l + 1] - offsets[l])
        ref = pipeline.decompress_layer(pay[offsets[l]:offsets[l] + size], n, int(batch.rows[l]),
                                        int(batch.cols[l]), cand)
        ref_acc = pipeline.decompress_layer(pay[offsets[l]:offsets[l] + size], n, int(batch.rows[l]),
                                            int(batch.cols[l]), cand, out=base[off:off + n])
        if cand[0] == W.LOWRANK:
            scale = max(np.linalg.norm(ref.astype(np.float64)), 1e-30)
            assert np.linalg.norm(got[off:off + n].astype(np.float64) - ref) <= fro_tol * scale, l
            assert np.linalg.norm(got_acc[off:off + n].astype(np.float64) - ref_acc) <= \
                fro_tol * max(np.linalg.norm(ref_acc.astype(np.float64)), 1e-30), l
        else:
            assert np.array_equal(got[off:off + n].view(np.uint32), ref.view(np.uint32)), (l, cand)
            assert np.array_equal(got_acc[off:off + n].view(np.uint32), ref_acc.view(np.uint32)), (l, cand)
    # elements outside the layers are not touched
    assert (got[~covered] == sentinel).all()
    h.close()


def _ragged(family_cands, values="student_t3", ef="normal0.1"):
    shapes = ((1,), (7,), (127,), (128,), (129,), (513, 3), (1000,), (65536 + 640 + 5,), (3, 5, 7), (131072,))
    return W.Workload("ragged", shapes, family_cands, 0, 100, values, ef, (-4.0, -2.0))


@pytest.mark.parametrize("stochastic", (False, True))
def test_quant_every_bit_width_ragged_layers(stochastic):
    w = _ragged(tuple((W.QUANT, float(b)) for b in range(1, 9)))
    batch = W.generate(w)
    L = len(batch.numels)
    for shift in range(3):
        choice = np.array([(l + shift * 3) % 8 for l in range(L)], np.int32)
        _roundtrip(w, batch, choice, stochastic=stochastic)


@pytest.mark.parametrize("bits", range(1, 9))
def test_quant_lengths_around_the_fetch_depth(bits):
    # a workgroup's round is 4096 elements of whole chunks, 1024 of a ragged end; then rounds of
    # 1024 and 256 with remainders of them.  The second half of the layers starts behind a single element.
    lengths = (512, 1024, 1536, 3584, 4096, 4608, 7680, 8192 + 512, 255 + 1024, 8191)
    shapes = tuple((n,) for n in lengths + (1 + -sum(lengths) % 4,) + lengths)
    w = W.Workload("lengths", shapes, ((W.QUANT, float(bits)),), 0, 100, "student_t3", "normal0.1", (-4.0, -2.0))
    _roundtrip(w, W.generate(w), np.zeros(len(shapes), np.int32))


def test_topk_ragged_layers_and_ties():
    w = _ragged(tuple((W.TOPK, d) for d in (0.001, 0.01, 0.1, 0.5, 1.0)), values="laplace", ef="same")
    batch = W.generate(w)
    batch.grads[:] = np.round(batch.grads * 2e3) / 2e3          # many equal magnitudes
    L = len(batch.numels)
    for shift in range(2):
        choice = np.array([(l + shift * 2) % 5 for l in range(L)], np.int32)
        _roundtrip(w, batch, choice)


def test_mixed_small_gpt2_shaped():
    full = W.workload("c4_gpt2_medium_mixed")
    shapes = tuple(W.gpt2_medium_shapes(layers=2, d=128, d_ff=512, vocab=1000, ctx=64))
    w = W.Workload("mixed_small", shapes, full.candidates, full.default, 400, full.values, full.ef, full.scale_exp)
    batch = W.generate(w)
    choice = np.array([(5 * l) % len(w.candidates) for l in range(len(batch.numels))], np.int32)
    _roundtrip(w, batch, choice)


def test_lowrank_transformer_subset():
    full = W.workload("c3_transformer_lm_lowrank")
    shapes = tuple(W.transformer_lm_shapes(layers=2, d=128, d_ff=512, vocab=1000)) + ((37, 53), (130, 70))
    w = W.Workload("lr_small", shapes, full.candidates, full.default, 400, full.values, full.ef, full.scale_exp,
                   only_2d=True)
    batch = W.generate(w)
    L = len(batch.numels)
    choice = np.array([l % len(w.candidates) for l in range(L)], np.int32)
    _roundtrip(w, batch, choice, fro_tol=1e-3)


@pytest.mark.parametrize("rank", (1, 7, 8, 9, 33, 63, 64))
def test_lowrank_reconstruction_at_tile_edges(rank):
    """Feedback and image at remainders of the 64 x 64 tiles, the column spans of 512 and the steps of 8 ranks."""
    from paper_2210_17357_amd import binding as B
    torch = torch_cuda()
    shapes = ((1, 1), (63, 65), (64, 64), (65, 63), (128, 512), (64, 513), (66, 511), (3, 641), (130, 1100), (700, 5))
    w = W.Workload("lr_edges", shapes, ((W.LOWRANK, float(rank)),), 0, 100, "lowrank64", "normal0.1", (-3.0, -1.0), r_max=64)
    batch = W.generate(w)
    L = len(batch.numels)
    choice = np.zeros(L, np.int32)
    # P and Q as the payload holds them are exact here; of the product and the sum with x every element is off by at
    # most (r + 2) 2^-24 (|P| |Q|^T + |x|), and with orthonormal columns || |P| |Q|^T || <= sqrt(r) ||x||
    tol = (rank + 2) * 2.0 ** -24 * (rank ** 0.5 + 1.0)
    layers, ctab = tables(batch, list(w.candidates))
    g, e, q = to_device(batch)
    h = B.Handle(int(batch.grads.size), L, 1, r_max=64)
    offsets = B.payload_layout(layers, ctab, choice)
    payload = torch.zeros(int(offsets[-1]) + 16, dtype=torch.uint8, device="cuda")
    h.compress(g, e, layers, ctab, choice, payload, offsets, q)
    pay, left = payload.cpu().numpy(), e.cpu().numpy()
    h.close()
    for l in range(L):
        o, n, m_, n_ = int(batch.offsets[l]), int(batch.numels[l]), int(batch.rows[l]), int(batch.cols[l])
        f = pay[offsets[l]:offsets[l] + 4 * (m_ + n_) * rank].view(np.float32).astype(np.float64)
        image = f[:m_ * rank].reshape(m_, rank) @ f[m_ * rank:].reshape(n_, rank).T
        x = (batch.grads[o:o + n] + batch.ef[o:o + n]).astype(np.float64)
        assert np.linalg.norm(left[o:o + n] - (x - image.ravel())) <= tol * np.linalg.norm(x), (l, shapes[l])
    _roundtrip(w, batch, choice, fro_tol=1e-4)
