"""GPU parity of the quantization compressor and its receiver over how a call deals tiles to
workgroups: one chunk each, several, or longer parts where most layers belong to another family.
The results do not depend on it."""
import numpy as np
import pytest

from oracle import pipeline
from paper_2210_17357_amd import workloads as W

from gpu_util import tables, to_device, torch_cuda

pytestmark = pytest.mark.gpu

# ends of chunks (512), of parts (512, 2048, 4096, 8192) and of tiles (8192 here), and one short of or past them
LENGTHS = (1, 511, 512, 513, 2047, 2048, 2049, 2560, 4096, 4097, 7680, 8191, 8192, 8193, 8704, 16384 + 2048 + 77, 3 * 8192 + 512)


@pytest.mark.parametrize("stochastic", (False, True))
@pytest.mark.parametrize("share", ("all", "most", "few"))
def test_parts_of_tiles(share, stochastic):
    from paper_2210_17357_amd import binding as B
    torch = torch_cuda()
    quantized = sum(LENGTHS)
    other = {"all": 0, "most": quantized // 4, "few": quantized}[share]
    shapes = tuple((n,) for n in LENGTHS) + (((other,),) if other else ())
    cands = ((W.QUANT, 3.0), (W.QUANT, 8.0), (W.QUANT, 4.0), (W.TOPK, 0.01))
    w = W.Workload("parts", shapes, cands, 0, 100, "student_t3", "normal0.1", (-4.0, -2.0))
    batch = W.generate(w)
    L = len(shapes)
    choice = np.array([l % 3 if l < len(LENGTHS) else 3 for l in range(L)], np.int32)
    layers, ctab = tables(batch, list(cands))
    g, e, _ = to_device(batch)
    h = B.Handle(int(batch.grads.size), L, len(cands), stochastic=stochastic, seed=9)
    offsets = B.payload_layout(layers, ctab, choice)
    payload = torch.zeros(int(offsets[-1]) + 16, dtype=torch.uint8, device="cuda")
    h.compress(g, e, layers, ctab, choice, payload, offsets)
    out = torch.full((int(batch.grads.size),), 7.0, device="cuda")
    acc = torch.full((int(batch.grads.size),), 0.125, device="cuda")
    h.decompress(payload, offsets, layers, ctab, choice, out, accumulate=False)
    h.decompress(payload, offsets, layers, ctab, choice, acc, accumulate=True)
    pay, ef, got, added = payload.cpu().numpy(), e.cpu().numpy(), out.cpu().numpy(), acc.cpu().numpy()
    for l in range(L):
        off, n = int(batch.offsets[l]), int(batch.numels[l])
        p_ref, e_ref, _ = pipeline.compress_layer(batch.grads, batch.ef, off, n, 0, 0, cands[choice[l]], l,
                                                  stochastic=stochastic, seed=9)
        assert np.array_equal(pay[offsets[l]:offsets[l] + p_ref.size], p_ref), l
        assert np.array_equal(ef[off:off + n].view(np.uint32), e_ref.view(np.uint32)), l
        image = pipeline.decompress_layer(p_ref, n, 0, 0, cands[choice[l]])
        assert np.array_equal(got[off:off + n].view(np.uint32), image.view(np.uint32)), l
        assert np.array_equal(added[off:off + n], image + np.float32(0.125)), l
    h.close()


def test_largest_tiles_give_what_the_smallest_do():
    """67 M elements are cut into tiles of 32768, a part of them alone into tiles of 8192."""
    from paper_2210_17357_amd import binding as B
    torch = torch_cuda()
    n = (1 << 26) + 32768 + 8192 + 512 + 77
    gen = torch.Generator(device="cuda").manual_seed(3)
    g = torch.empty(n, device="cuda").normal_(generator=gen)
    e = torch.empty(n, device="cuda").normal_(generator=gen)
    ctab = B.cand_table([(W.QUANT, 5.0)])
    choice = np.zeros(1, np.int32)

    def run(lo, hi):
        layers = B.layer_table([0], [hi - lo], [0], [0])
        offsets = B.payload_layout(layers, ctab, choice)
        payload = torch.zeros(int(offsets[-1]) + 16, dtype=torch.uint8, device="cuda")
        h = B.Handle(hi - lo, 1, 1)
        ef, out = e[lo:hi].clone(), torch.zeros(hi - lo, device="cuda")
        h.compress(g[lo:hi].clone(), ef, layers, ctab, choice, payload, offsets)
        h.decompress(payload, offsets, layers, ctab, choice, out, accumulate=False)
        h.close()
        return ef, out

    ef, out = run(0, n)
    for lo in (0, 1 << 24, (1 << 26) - 65536):                 # whole buckets
        hi = min(lo + 4_000_000 // 128 * 128, n)
        ef_part, out_part = run(lo, hi)
        assert torch.equal(ef[lo:hi], ef_part) and torch.equal(out[lo:hi], out_part), lo


@pytest.mark.parametrize("stochastic", (False, True))
@pytest.mark.parametrize("n", ((1 << 26) + 4096 + 512 + 77, (1 << 24) + 8192 + 4096 - 512, (1 << 24) + (1 << 20) + 3))
def test_profile_of_parts_adds_up(n, stochastic):
    """Tiles of 32768 and 16384 elements are profiled in parts; pieces of the same data in a handle of their own have
    tiles of 8192.  Buckets are the same, so with deterministic rounding the errors add up to the whole's; the numbers
    of stochastic rounding depend on the place in the layer, so there the first piece alone is compared, cut short."""
    from paper_2210_17357_amd import binding as B
    torch = torch_cuda()
    gen = torch.Generator(device="cuda").manual_seed(4)
    g = torch.empty(n, device="cuda").normal_(generator=gen)
    cands = [(W.QUANT, 2.0), (W.QUANT, 4.0), (W.QUANT, 7.0)]
    ctab = B.cand_table(cands)

    def profile(x, lengths):
        offs = np.concatenate([[0], np.cumsum(lengths)[:-1]])
        layers = B.layer_table(offs, lengths, [0] * len(lengths), [0] * len(lengths))
        h = B.Handle(int(x.numel()), len(lengths), 3, stochastic=stochastic, seed=11)
        errors, _ = h.profile(x, None, layers, ctab)
        h.close()
        return errors

    whole = profile(g, [n])
    step = 1 << 22
    if stochastic:
        # layers of one handle: the first holds the same elements at the same places
        split = profile(g, [step, n - step])
        alone = profile(g[:step].clone(), [step])
        assert np.allclose(split[0], alone[0], rtol=1e-6) and (whole[0] > split[0]).all()
        return
    parts = sum(profile(g[lo:min(lo + step, n)].clone(), [min(step, n - lo)])[0] for lo in range(0, n, step))
    # fp32 sums of at most 64 squares a lane, then fp64
    assert np.allclose(whole[0], parts, rtol=64 * 2.0 ** -24), (whole, parts)
