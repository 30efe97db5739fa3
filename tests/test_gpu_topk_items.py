"""GPU parity of Top-K where the refinement has more work items than start at once: they run in another order than
that of the layers."""
import numpy as np
import pytest

from oracle import pipeline
from paper_2210_17357_amd import workloads as W

from gpu_util import rel_err, tables, tile_size, to_device, torch_cuda

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("densities", ((0.01,), (0.001, 0.01, 0.1), tuple(i / 100 for i in range(1, 13))))
@pytest.mark.parametrize("n_layers", (511, 513, 700))
def test_more_items_than_slots(n_layers, densities):
    from paper_2210_17357_amd import binding as B
    torch = torch_cuda()
    rng = np.random.default_rng(n_layers)
    sizes = rng.integers(1, 3000, n_layers)
    sizes[::97] = rng.integers(8000, 40000, sizes[::97].size)       # several tiles, among layers of one
    w = W.Workload("items", tuple((int(n),) for n in sizes), tuple((W.TOPK, d) for d in densities), 0, 100, "laplace",
                   "normal0.1", (-4.0, -2.0))
    batch = W.generate(w)
    cands = list(w.candidates)
    layers, ctab = tables(batch, cands)
    g, e, _ = to_device(batch)
    h = B.Handle(int(batch.grads.size), n_layers, len(cands))
    errors, _ = h.profile(g, e, layers, ctab)
    ref = pipeline.profile(batch.grads, batch.ef, batch.offsets, batch.numels, batch.rows, batch.cols, cands)
    assert ((rel_err(errors, ref) < 1e-4) | (np.abs(errors - ref) < 1e-30)).all()
    again, _ = h.profile(g, e, layers, ctab)
    assert np.array_equal(errors, again)
    choice = np.full(n_layers, len(cands) - 1, np.int32)
    offsets = B.payload_layout(layers, ctab, choice)
    payload = torch.zeros(int(offsets[-1]) + 16, dtype=torch.uint8, device="cuda")
    h.compress(g, e, layers, ctab, choice, payload, offsets)
    pay = payload.cpu().numpy()
    for l in range(0, n_layers, 7):
        p_ref, _, _ = pipeline.compress_layer(batch.grads, batch.ef, int(batch.offsets[l]), int(batch.numels[l]), 0, 0,
                                              cands[choice[l]], l)
        assert np.array_equal(pay[offsets[l]:offsets[l] + p_ref.size], p_ref), l
    h.close()


def test_lists_of_both_kinds_take_turns_on_one_handle():
    """At 18 M elements a call with Top-K layers cuts them into tiles of 16384, one without into tiles of 8192: on one handle,
    behind profiles of every kind of list, profiles and compressions give what a handle of their own gives, bit for
    bit, and layers alone (tiles of 8192) the same payload as in the table."""
    from paper_2210_17357_amd import binding as B
    torch = torch_cuda()
    sizes = [9_000_000, 5_000_001, 77, 4_000_000 - 512, 16384, 8193]
    offs = np.concatenate([[0], np.cumsum(sizes)[:-1]])
    total, n = sum(sizes), len(sizes)
    assert tile_size(total, True) == 16384 and tile_size(total, False) == 8192
    gen = torch.Generator(device="cuda").manual_seed(8)
    g = torch.empty(total, device="cuda").normal_(generator=gen)
    e = torch.empty(total, device="cuda").normal_(generator=gen)
    layers = B.layer_table(offs, sizes, [0] * n, [0] * n)
    cands = [(W.QUANT, 3.0), (W.QUANT, 6.0), (W.TOPK, 0.01), (W.TOPK, 0.1)]
    ctab = B.cand_table(cands)
    lists = [B.cand_table(cands[:2]), ctab, B.cand_table(cands[2:])]
    choices = [np.array(c, np.int32) for c in ((0, 1, 0, 1, 0, 1), (0, 2, 3, 1, 2, 0), (2, 3, 2, 2, 3, 3))]

    def compress(h, table, choice, lo=0, hi=total):
        offsets = B.payload_layout(table, ctab, choice)
        payload, ef = torch.zeros(int(offsets[-1]) + 16, dtype=torch.uint8, device="cuda"), e[lo:hi].clone()
        h.compress(g[lo:hi].clone(), ef, table, ctab, choice, payload, offsets)
        out = torch.zeros(hi - lo, device="cuda")
        h.decompress(payload, offsets, table, ctab, choice, out, accumulate=False)
        return offsets, payload, ef, out

    shared = B.Handle(total, n, 4)
    for choice in choices:
        own = B.Handle(total, n, 4)
        offsets, *want = compress(own, layers, choice)
        own.close()
        for profiled in lists:                              # of the compression's kind and of the others
            own = B.Handle(total, n, 4)
            assert np.array_equal(shared.profile(g, e, layers, profiled)[0], own.profile(g, e, layers, profiled)[0])
            own.close()
            _, *got = compress(shared, layers, choice)
            assert all(torch.equal(a, b) for a, b in zip(want, got))
        for l in (1, 2, 3, 5):
            lo, hi = int(offs[l]), int(offs[l]) + sizes[l]
            alone = B.Handle(sizes[l], 1, 4)
            one = compress(alone, B.layer_table([0], [sizes[l]], [0], [0]), choice[l:l + 1], lo, hi)
            alone.close()
            size = int(B.sizes(layers, ctab)[l, choice[l]])
            assert torch.equal(want[0][int(offsets[l]):int(offsets[l]) + size], one[1][:size]), l
            assert torch.equal(want[1][lo:hi], one[2]) and torch.equal(want[2][lo:hi], one[3]), l
    shared.close()


def test_calls_of_both_kinds_leave_each_other_nothing_to_upload():
    """Calls with Top-K layers and calls without keep a cut of the layers on the device each: whatever calls come between,
    a compression that ran before queues kernels alone, so that it can be captured, and gives on every replay what a handle of
    its own gives."""
    from paper_2210_17357_amd import binding as B
    torch = torch_cuda()
    sizes = [9_000_000, 5_000_001, 77, 4_000_000 - 512, 16384, 8193]
    offs = np.concatenate([[0], np.cumsum(sizes)[:-1]])
    total, n = sum(sizes), len(sizes)
    gen = torch.Generator(device="cuda").manual_seed(8)
    g = torch.empty(total, device="cuda").normal_(generator=gen)
    e = torch.empty(total, device="cuda").normal_(generator=gen)
    layers = B.layer_table(offs, sizes, [0] * n, [0] * n)
    quant, both = B.cand_table([(W.QUANT, 3.0)]), B.cand_table([(W.QUANT, 3.0), (W.TOPK, 0.01), (W.TOPK, 0.1)])
    choices = np.zeros(n, np.int32), np.array([0, 1, 2, 1, 0, 2], np.int32)
    layouts = [B.payload_layout(layers, both, c) for c in choices]

    def buffers():
        return e.clone(), torch.zeros(int(layouts[0][-1]) + 16, dtype=torch.uint8, device="cuda")

    h, own = B.Handle(total, n, 3), B.Handle(total, n, 3)
    ef, payload = buffers()
    stream = torch.cuda.Stream()

    def profiles():
        h.profile(g, e, layers, quant)
        h.profile(g, e, layers, both)

    for choice, offsets in zip(choices, layouts):
        h.compress(g, ef, layers, both, choice, payload, offsets)
        profiles()
    graphs = []
    for choice, offsets in zip(choices, layouts):
        torch.cuda.synchronize()
        graphs.append(torch.cuda.CUDAGraph())
        with torch.cuda.graph(graphs[-1], stream=stream):
            h.compress(g, ef, layers, both, choice, payload, offsets, stream=stream.cuda_stream)
        profiles()
    ef.copy_(e)
    want_ef, want_payload = buffers()
    for _ in range(3):
        for graph, choice, offsets in zip(graphs, choices, layouts):
            payload.zero_()
            want_payload.zero_()
            torch.cuda.synchronize()
            graph.replay()
            own.compress(g, want_ef, layers, both, choice, want_payload, offsets)
            torch.cuda.synchronize()
            assert torch.equal(ef, want_ef) and torch.equal(payload, want_payload)
            profiles()
    del graphs
    h.close()
    own.close()
