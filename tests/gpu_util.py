"""Helpers for the GPU parity tests: move a synthetic batch to the device and call the C ABI
through the binding."""
import numpy as np


def torch_cuda():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    return torch


def to_device(batch):
    torch = torch_cuda()
    g = torch.from_numpy(batch.grads).cuda()
    e = None if batch.ef is None else torch.from_numpy(batch.ef).cuda()
    q = None if batch.q0 is None else torch.from_numpy(batch.q0).cuda()
    return g, e, q


def tables(batch, cands):
    from paper_2210_17357_amd import binding as B
    return (B.layer_table(batch.offsets, batch.numels, batch.rows, batch.cols), B.cand_table(cands))


def rel_err(a, b):
    a = np.asarray(a, np.float64)
    b = np.asarray(b, np.float64)
    return np.abs(a - b) / np.maximum(np.abs(b), 1e-300)


def tile_size(total, topk):
    """Tile size of a layer table of `total` elements in calls with and without Top-K layers (checked against the library's
    rule by test_parts_rule)."""
    tile = 32768
    while tile > 8192 and total // tile < (1024 if topk and tile < 32768 else 2048):
        tile //= 2
    return tile


def many_small(n_layers):
    """Lengths of so many layers, most below 1500 elements, that parts of tiles are longer than asked for: 4096 elements of
    tiles of 8192 for 1200 layers, whole tiles for 3000."""
    rng = np.random.default_rng(n_layers)
    lengths = rng.integers(1, 1500, n_layers)
    lengths[::300] = rng.integers(8192, 40000, lengths[::300].size)
    lengths[7:n_layers:400] = 8192 + 4096 + 512 + 3
    return lengths


def tile_count(lengths, tile):
    n = np.asarray(lengths, np.int64)
    rest = n % tile
    return int((n // tile + (rest >= 512) + (rest % 512 > 0)).sum())
