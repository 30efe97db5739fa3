"""GPU parity of the quantization profile, compressor and receiver over how a table is cut into tiles and how a call deals
tiles to workgroups: one chunk each, several, or longer parts where most layers belong to another family or are small.
The results do not depend on it."""
import numpy as np
import pytest

from oracle import pipeline
from paper_2210_17357_amd import workloads as W

from gpu_util import many_small, tables, tile_size, to_device, torch_cuda

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


def _check_layer(batch_g, batch_e, l, off, n, cand, pay, ef, got, stochastic, seed):
    p_ref, e_ref, _ = pipeline.compress_layer(batch_g, batch_e, off, n, 0, 0, cand, l, stochastic=stochastic, seed=seed)
    assert np.array_equal(pay[:p_ref.size], p_ref), l
    assert np.array_equal(ef[off:off + n].view(np.uint32), e_ref.view(np.uint32)), l
    assert np.array_equal(got[off:off + n].view(np.uint32), pipeline.decompress_layer(p_ref, n, 0, 0, cand).view(np.uint32)), l


@pytest.mark.parametrize("stochastic", (False, True))
@pytest.mark.parametrize("n_layers", (1200, 3000))
def test_many_small_layers(n_layers, stochastic):
    """So many tiles that are not full that parts are 4096 elements (1200 layers) or whole tiles (3000)."""
    from paper_2210_17357_amd import binding as B
    torch = torch_cuda()
    lengths = many_small(n_layers)
    offs = np.concatenate([[0], np.cumsum(lengths)[:-1]])
    total = int(lengths.sum())
    rng = np.random.default_rng(21)
    g, e = (rng.standard_normal(total).astype(np.float32) for _ in range(2))
    cands = [(W.QUANT, 5.0), (W.QUANT, 2.0), (W.TOPK, 0.05)]
    layers, ctab = B.layer_table(offs, lengths, [0] * n_layers, [0] * n_layers), B.cand_table(cands)
    h = B.Handle(total, n_layers, 3, stochastic=stochastic, seed=13)
    for few in (False, True):
        choice = (np.arange(n_layers) % (3 if few else 2)).astype(np.int32)
        offsets = B.payload_layout(layers, ctab, choice)
        payload = torch.zeros(int(offsets[-1]) + 16, dtype=torch.uint8, device="cuda")
        ef, out = torch.from_numpy(e).cuda(), torch.full((total,), 7.0, device="cuda")
        h.compress(torch.from_numpy(g).cuda(), ef, layers, ctab, choice, payload, offsets)
        h.decompress(payload, offsets, layers, ctab, choice, out, accumulate=False)
        pay, left, got = payload.cpu().numpy(), ef.cpu().numpy(), out.cpu().numpy()
        for l in sorted(set(range(0, n_layers, 41)) | set(range(0, n_layers, 300)) | set(range(7, n_layers, 400))):
            _check_layer(g, e, l, int(offs[l]), int(lengths[l]), cands[choice[l]], pay[offsets[l]:], left, got, stochastic, 13)
    h.close()


@pytest.mark.parametrize("stochastic", (False, True))
@pytest.mark.parametrize("total,tile", ((1 << 24, 16384), ((1 << 26) + 77, 32768)))
def test_parts_of_larger_tiles_beside_another_family(total, tile, stochastic):
    """Most elements belong to a Top-K layer, so quantized tiles are dealt to workgroups of 8192 elements, two or four a
    tile; ends around those parts and around tiles."""
    from paper_2210_17357_amd import binding as B
    torch = torch_cuda()
    assert tile_size(total, True) == tile
    ends = (8192, tile // 2, tile - 512, tile)
    lengths = [k * tile + n + d for k in (0, 1) for n in ends for d in (-512, -1, 0, 1, 512)] + [1, 100, 511]
    lengths.insert(5, total - sum(lengths))
    big, L = 5, len(lengths)
    offs = np.concatenate([[0], np.cumsum(lengths)[:-1]])
    gen = torch.Generator(device="cuda").manual_seed(31)
    g = torch.empty(total, device="cuda").normal_(generator=gen)
    e = torch.empty(total, device="cuda").normal_(generator=gen)
    cands = [(W.QUANT, 5.0), (W.QUANT, 8.0), (W.QUANT, 3.0), (W.TOPK, 0.001)]
    choice = np.array([3 if l == big else l % 3 for l in range(L)], np.int32)
    layers, ctab = B.layer_table(offs, lengths, [0] * L, [0] * L), B.cand_table(cands)
    h = B.Handle(total, L, 4, stochastic=stochastic, seed=17)
    offsets = B.payload_layout(layers, ctab, choice)
    payload = torch.zeros(int(offsets[-1]) + 16, dtype=torch.uint8, device="cuda")
    ef, out, acc = e.clone(), torch.full((total,), 7.0, device="cuda"), g.clone()
    h.compress(g, ef, layers, ctab, choice, payload, offsets)
    h.decompress(payload, offsets, layers, ctab, choice, out, accumulate=False)
    h.decompress(payload, offsets, layers, ctab, choice, acc, accumulate=True)
    h.close()
    assert torch.equal(acc, g + out)
    pay, left, got, hg, he = payload.cpu().numpy(), ef.cpu().numpy(), out.cpu().numpy(), g.cpu().numpy(), e.cpu().numpy()
    for l in range(L):
        if l != big:
            _check_layer(hg, he, l, int(offs[l]), lengths[l], cands[choice[l]], pay[offsets[l]:], left, got, stochastic, 17)
    # the Top-K layer: the largest magnitudes go, the rest stays
    x = (hg + he)[offs[big]:offs[big] + lengths[big]]
    part, image = left[offs[big]:offs[big] + lengths[big]], got[offs[big]:offs[big] + lengths[big]]
    sent = image != 0
    assert sent.sum() == int(0.001 * lengths[big] + 0.5) and np.array_equal(image[sent], x[sent])
    assert np.array_equal(part[~sent], x[~sent]) and not part[sent].any()
    assert np.abs(x[sent]).min() >= np.abs(x[~sent]).max()


@pytest.mark.parametrize("stochastic", (False, True))
def test_profile_does_not_depend_on_the_size_of_tiles(stochastic):
    """The first layer's errors, with a second one that makes the tiles 8192, 16384 and 32768 elements: the oracle's,
    whose numbers of stochastic rounding follow the place in the layer as well."""
    from paper_2210_17357_amd import binding as B
    torch = torch_cuda()
    n = (1 << 20) + 8192 + 512 + 77
    totals = {8192: n + (1 << 20), 16384: (1 << 25) + 3, 32768: (1 << 26) + 5}
    gen = torch.Generator(device="cuda").manual_seed(4)
    g = torch.empty(max(totals.values()), device="cuda").normal_(generator=gen)
    cands = [(W.QUANT, 2.0), (W.QUANT, 4.0), (W.QUANT, 7.0)]
    ctab = B.cand_table(cands)
    ref = pipeline.profile(g[:n].cpu().numpy(), None, [0], [n], [0], [0], cands, stochastic=stochastic, seed=11)
    for tile, total in totals.items():
        assert tile_size(total, False) == tile
        layers = B.layer_table([0, n], [n, total - n], [0, 0], [0, 0])
        h = B.Handle(total, 2, 3, stochastic=stochastic, seed=11)
        errors, _ = h.profile(g, None, layers, ctab)
        h.close()
        # fp32 sums of at most 128 squares a lane (the largest tile over 256 lanes), in fp64 from there
        assert np.allclose(errors[0], ref[0], rtol=128 * 2.0 ** -24, atol=0), (tile, errors[0], ref[0])
