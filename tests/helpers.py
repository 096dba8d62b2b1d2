"""Shared plumbing of the GPU parity tests: build the HIP context and the oracle from the
same description, move seeded inputs to the device, compare."""
from __future__ import annotations

import numpy as np

from oracle import accordion_oracle as orc
from paper_2010_16248_amd import binding as B


def layer_tuples(layers):
    return [(l.offset, l.rows, l.cols, l.is_matrix) if hasattr(l, "offset") else tuple(l) for l in layers]


def make_pair(method, layers, W, crit, noncrit, k_den=100, eta=0.5, initial_level=1, q_init=None):
    lt = layer_tuples(layers)
    gpu = B.Accordion(method, lt, W, crit, noncrit, k_den, eta, initial_level, q_init)
    ora = orc.AccordionOracle(method, lt, W, crit, noncrit, k_den, eta, initial_level, q_init)
    return gpu, ora


def make_pair_in(n, method, layers, *args):
    """make_pair in flat buffers of n elements: the layers, elements of no layer, and a last layer of four that ends at n.  A
    context of any size for the work of a small one.  ora.inside: the elements that belong to a layer; the others of an
    output buffer are not written."""
    lt = layer_tuples(layers) + [(n - 4, 1, 4, 0)]
    gpu, ora = make_pair(method, lt, *args)
    assert gpu.n_params == n
    ora.N, ora.e, ora.A = n, np.zeros((ora.W, n), np.float32), np.zeros(n, np.float32)
    ora.inside = np.zeros(n, bool)
    for off, rows, cols, _ in lt:
        ora.inside[off:off + rows * cols] = True
    return gpu, ora


def in_buffer(values, n):
    """values at the start of a flat buffer of n elements, the rest zero."""
    out = np.zeros(n, np.float32)
    out[:values.size] = values
    return out


def to_dev(a):
    import torch
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda:0")


def dev_out(n):
    import torch
    return torch.empty(n, dtype=torch.float32, device="cuda:0")


def bits(a):
    return np.ascontiguousarray(a, dtype=np.float32).view(np.uint32)


def assert_bits_equal(got, ref, what=""):
    g, r = bits(got), bits(ref)
    if not np.array_equal(g, r):
        bad = np.flatnonzero(g != r)
        raise AssertionError(f"{what}: {bad.size} of {g.size} words differ, first at {bad[0]}: "
                             f"{np.asarray(got).reshape(-1)[bad[0]]!r} vs {np.asarray(ref).reshape(-1)[bad[0]]!r}")


def rel_fro(got, ref):
    got = np.asarray(got, np.float64)
    ref = np.asarray(ref, np.float64)
    den = np.linalg.norm(ref)
    num = np.linalg.norm(got - ref)
    return num / den if den > 0 else num


def oracle_state_blob(gpu, ora):
    """The oracle's state in the library's state layout (teacher forcing)."""
    q = np.concatenate([ora.Q[li].reshape(-1) for li in sorted(ora.Q)]) if ora.Q else np.zeros(0, np.float32)
    return gpu.pack_state(ora.e, ora.A, q, ora.norm_old, ora.has_old, ora.level)


def powersgd_workspace_bytes(layers, W, rmax, rows_first, rows_right):
    """accordion_workspace_bytes of a PowerSGD configuration whose matrix tiles have rows_first rows (first pass,
    decompression) and rows_right rows (right product), region by region: tells which tiles a configuration got."""
    lt = layer_tuples(layers)
    end = max(off + r * c for off, r, c, _ in lt)
    N64 = (end + 63) // 64 * 64
    mats = [(r, c) for _, r, c, m in lt if m]

    def up(a, b):
        return -(-a // b)

    def tiles(rows):
        return sum(up(r, rows) * up(c, 256) for r, c in mats)

    nl, flat = len(lt), sum(up(r * c, 8192) for _, r, c, _ in lt)
    p_total = sum(r for r, _ in mats) * rmax
    regions = [120 * nl, 16 * flat, 16 * tiles(rows_first), 16 * tiles(rows_right), 8 * sum(up(c, 256) for _, c in mats),
               8 * sum(up(r, 16) for r, _ in mats), 4 * sum(up(r * c, 8192) for _, r, c, m in lt if not m), 4 * len(mats)]
    regions += [4 * nl] * 6 + [48, 4 * N64, 4 * N64 * W, 8 * flat, 8 * tiles(rows_first), 4, 0, 32]
    regions += [16 * sum(c for _, c in mats), 4 * p_total, 8 * p_total, 8 * W * rmax * sum(r * up(c, 256) for r, c in mats),
                8 * W * rmax * sum(c * up(r, rows_right) for r, c in mats), 4 * sum(r * c for _, r, c, m in lt if not m), 4]
    return sum(up(b, 256) * 256 for b in regions)
