"""GPU parity: TopK with error feedback against the oracle, bit for bit, through the C ABI."""
import numpy as np
import pytest

from oracle import accordion_oracle as orc
from paper_2010_16248_amd import binding as B
from paper_2010_16248_amd import workloads as wl
from tests import helpers as H

pytestmark = pytest.mark.gpu


def _check_step(gpu, ora, grads, tag, check_state=True):
    """One batched step on both sides; mean and payloads always compared.  check_state=False
    leaves the library's memory alone (reading it writes the residual out, which the batched
    path otherwise defers to the next step's first pass): the deferred route is then the one
    the next step takes.  Returns the mean."""
    out_ref = ora.step(grads)
    dg = [H.to_dev(g) for g in grads]
    out = H.dev_out(gpu.n_params)
    gpu.step_all(dg, out)
    mean = out.cpu().numpy()
    inside = getattr(ora, "inside", slice(None))
    H.assert_bits_equal(mean[inside], out_ref[inside], f"{tag}: mean")
    for w in range(gpu.n_workers):
        for li in range(gpu.n_layers):
            idx, val = gpu.get_payload(w, li)
            ri, rv = ora.payload[(w, li)]
            assert np.array_equal(idx, ri), f"{tag}: indices worker {w} layer {li}"
            H.assert_bits_equal(val, rv, f"{tag}: values worker {w} layer {li}")
    assert gpu.payload_words() == (ora.words_last, ora.words_cum)
    if not check_state:
        return mean
    st = gpu.unpack_state(gpu.get_state())
    H.assert_bits_equal(st["e"], ora.e, f"{tag}: residual")
    H.assert_bits_equal(st["A"], ora.A, f"{tag}: accumulator")
    return mean


def _case_values(rng, case, n):
    if case == "normal":
        return rng.standard_normal(n)
    if case == "quantised":
        return rng.integers(-3, 4, n) * 0.25
    if case == "all_equal":
        return np.full(n, -1.5)
    if case == "all_zero":
        return np.zeros(n)
    if case == "sparse":
        return rng.standard_normal(n) * (rng.random(n) < 0.05)
    raise KeyError(case)


@pytest.mark.parametrize("W", [1, 3])
def test_kept_entries_concentrated_in_a_few_quarters(W):
    """K = 25 % and 45 % of layers whose large entries sit in one stretch: whole wave quarters
    are kept, so a wave's list of payload entries fills up inside a chunk of groups and is
    written out early, while other quarters keep nothing.  Aligned and misaligned layers, the
    stretch at a different place for every worker."""
    print(f"case concentrated W={W}", flush=True)
    shapes = [(1, 5 * 8192, 0), (1, 3, 0), (3, 8192 + 1001, 1), (1, 2 * 8192 + 6, 0)]
    layers = wl.make_layers(shapes)
    N = wl.total_params(layers)
    gpu, ora = H.make_pair(B.ACC_TOPK, layers, W, 45, 25)
    rng = np.random.default_rng(77 + W)
    for step in range(4):
        if step == 2:
            ora.level[:] = 0
            gpu.set_state(H.oracle_state_blob(gpu, ora))
        grads = []
        for w in range(W):
            g = rng.standard_normal(N) * 1e-3
            for l in layers:
                n = l.numel
                lo = (n // 7) * ((w + step) % 5)
                hi = min(n, lo + int(n * 0.4))
                g[l.offset + lo:l.offset + hi] += np.sign(rng.standard_normal(hi - lo)) * (1.0 + rng.random(hi - lo))
            grads.append(g.astype(np.float32))
        _check_step(gpu, ora, grads, f"step {step}", check_state=(step % 2 == 1))
    gpu.destroy()


@pytest.mark.parametrize("crit,noncrit,den", [(10, 1, 100), (1, 1, 1), (1, 3, 1000), (99, 25, 100)])
def test_ragged_misaligned_layers(crit, noncrit, den):
    """Many small layers at 16-byte-misaligned offsets, W = 3, several steps so that the
    memory feeds back; K from 0.1 % to 100 %."""
    print(f"case ragged crit={crit} noncrit={noncrit} den={den}", flush=True)
    layers = wl.random_layers(seed=11, n_layers=23, max_rows=40, max_cols=300)
    N = wl.total_params(layers)
    gpu, ora = H.make_pair(B.ACC_TOPK, layers, 3, crit, noncrit, den)
    rng = np.random.default_rng(1)
    for step in range(3):
        grads = [rng.standard_normal(N).astype(np.float32) for _ in range(3)]
        _check_step(gpu, ora, grads, f"step {step}", check_state=(step == 2))
    # switch every layer to the other level by hand and go on
    blob = H.oracle_state_blob(gpu, ora)
    ora.level[:] = 0
    st = gpu.unpack_state(blob)
    st["level"][:] = 0
    gpu.set_state(blob)
    for step in range(2):
        grads = [rng.standard_normal(N).astype(np.float32) for _ in range(3)]
        _check_step(gpu, ora, grads, f"noncrit step {step}", check_state=(step == 1))
    gpu.destroy()


@pytest.mark.parametrize("case", ["normal", "quantised", "all_equal", "all_zero", "sparse"])
def test_multi_tile_layers_with_ties(case):
    """Layers that span several 8192-element tiles with ragged tails; value sets with heavy
    ties (the lower index must win) including a tie class far larger than the candidate
    list, which takes the re-read path."""
    print(f"case multi-tile {case}", flush=True)
    shapes = [(1, 3 * 8192 + 77, 0), (37, 1001, 1), (1, 5, 0), (3, 8192, 1), (1, 70001, 0)]
    layers = wl.make_layers(shapes)
    N = wl.total_params(layers)
    gpu, ora = H.make_pair(B.ACC_TOPK, layers, 2, 10, 1)
    rng = np.random.default_rng([7, len(case)])
    for step in range(4):                                    # state read after steps 1 and 3 only
        grads = [_case_values(rng, case, N).astype(np.float32) for _ in range(2)]
        _check_step(gpu, ora, grads, f"{case} step {step}", check_state=(step % 2 == 1))
    gpu.destroy()


@pytest.mark.parametrize("W", [2, 3, 4, 8])
def test_mean_of_subnormal_values_rounds_like_a_division(W):
    """Kept values so small that their mean is subnormal: the mean must round exactly like the
    oracle's division by W (for W a power of two the kernel multiplies by 1 / W, which is the same
    real number), over several steps so that subnormal residuals feed back as well."""
    print(f"case subnormal mean W={W}", flush=True)
    layers = wl.make_layers([(1, 2 * 8192 + 31, 0), (9, 333, 1)])
    N = wl.total_params(layers)
    gpu, ora = H.make_pair(B.ACC_TOPK, layers, W, 50, 10)
    rng = np.random.default_rng([13, W])
    tiny = np.float32(1.4e-45)
    for step in range(3):
        grads = [(rng.integers(-40, 41, N).astype(np.float32) * tiny) for _ in range(W)]
        assert all(np.all(np.abs(g) < 1.2e-38) for g in grads)
        _check_step(gpu, ora, grads, f"subnormal W={W} step {step}", check_state=(step == 2))
    gpu.destroy()


def test_guessed_bins_hit_drift_and_miss():
    """The error-feedback pass lists its candidates on a guess of where the threshold will lie.
    Over many steps with a stationary distribution the guess must hit (nothing is staged again, the
    compaction works from the lists); a slow drift of the gradient scale is followed by the
    extrapolated guess; a jump makes it miss (the layer is staged again and compacted from Delta).
    Every step is bit-exact whichever route is taken -- against the oracle, and word for word
    against a second context that is driven call by call, where the compaction always reads
    Delta and the mean is formed from the payloads."""
    print("case guessed bins", flush=True)
    shapes = [(1, 5 * 8192 + 13, 0), (64, 577, 1), (1, 100, 0), (6, 8192, 1)]
    layers = wl.make_layers(shapes)
    N = wl.total_params(layers)
    W = 2
    gpu, ora = H.make_pair(B.ACC_TOPK, layers, W, 10, 1)
    twin, _ = H.make_pair(B.ACC_TOPK, layers, W, 10, 1)
    out_twin = H.dev_out(N)
    rng = np.random.default_rng(5)
    scale = 1.0
    restaged = []
    for step in range(14):
        if 6 <= step < 10:
            scale *= 1.09                                   # one level-1 bin per step, about
        if step == 12:
            scale *= 40.0                                   # far outside the guessed bins
        grads = [(rng.standard_normal(N) * scale).astype(np.float32) for _ in range(W)]
        mean = _check_step(gpu, ora, grads, f"step {step}", check_state=(step % 3 == 2 or step == 13))
        restaged.append(gpu.topk_stats()[0])
        dg = [H.to_dev(g) for g in grads]
        for w in range(W):
            twin.compress_step(w, dg[w], 0)
        twin.aggregate(0)
        twin.decompress(out_twin)
        H.assert_bits_equal(out_twin.cpu().numpy(), mean, f"step {step}: the two routes differ in the mean")
        for w in range(W):
            for li in range(gpu.n_layers):
                ia, va = gpu.get_payload(w, li)
                ib, vb = twin.get_payload(w, li)
                assert np.array_equal(ia, ib), f"step {step}: the two routes differ in the indices"
                H.assert_bits_equal(va, vb, f"step {step}: the two routes differ in the values")
    per_step = np.diff([0] + restaged)
    n_multi = 3 * W                                         # (worker, layer) pairs of more than one tile
    assert per_step[0] == n_multi                           # nothing to guess from at the first step
    assert per_step[3:6].sum() == 0, per_step               # stationary: the guess holds
    assert per_step[12] == n_multi, per_step                # the jump is missed ...
    assert per_step[13] <= n_multi                          # ... and everything is still exact
    assert gpu.topk_stats()[1] == 0                         # no tie class needed the sweeps
    twin.destroy()
    gpu.destroy()


def test_a_level_switch_finds_its_bins_guessed_from_the_other_level():
    """While a level runs, the bins of the other level's threshold are taken from the same
    histogram, so the first step after a switch needs no second staging on a stationary
    distribution (its own history at that level is missing or stale); results stay bit-exact."""
    print("case level switch guess", flush=True)
    shapes = [(1, 5 * 8192 + 13, 0), (64, 577, 1), (1, 100, 0), (6, 8192, 1)]
    layers = wl.make_layers(shapes)
    N = wl.total_params(layers)
    W = 2
    gpu, ora = H.make_pair(B.ACC_TOPK, layers, W, 10, 1)
    rng = np.random.default_rng(15)
    restaged = []
    for step in range(12):
        if step in (2, 4, 8):                               # windows of 2, 2 and 4 steps
            # no history: critical (K 10 % stays); stationary norms: non-critical (K 1 % from step
            # 4); a learning-rate decay: critical (K 10 % again from step 8)
            lr_next = 0.01 if step == 8 else 0.1
            ref = ora.detect_regime(0.1, lr_next)
            gpu.detect_regime(0.1, lr_next)
            assert np.array_equal(gpu.get_levels(), ref)
        grads = [rng.standard_normal(N).astype(np.float32) for _ in range(W)]
        _check_step(gpu, ora, grads, f"step {step}", check_state=(step % 4 == 3))
        restaged.append(gpu.topk_stats()[0])
    per_step = np.diff([0] + restaged)
    assert per_step[0] == 3 * W                             # nothing to guess from at the very first step
    assert ora.level[0] == 1 and ora.words_cum > 0
    assert per_step[4] == 0 and per_step[8] == 0, per_step  # the first steps at a new level
    gpu.destroy()


def test_threshold_among_exact_zeros_is_guessed_too():
    """Sparse gradients of which more is kept than is non-zero (the embedding of a language
    model): the threshold is zero.  After the first step the error-feedback pass stages bin 0
    itself (non-zero keys listed, zeros counted), so nothing is re-staged; a dense step in
    between is a miss and everything stays exact."""
    print("case zero-bin guess", flush=True)
    shapes = [(1, 5 * 8192 + 13, 0), (64, 577, 1)]
    layers = wl.make_layers(shapes)
    N = wl.total_params(layers)
    W = 2
    gpu, ora = H.make_pair(B.ACC_TOPK, layers, W, 10, 1)
    rng = np.random.default_rng(15)
    restaged = []
    for step in range(7):
        dense = step == 4
        grads = []
        for _ in range(W):
            g = rng.standard_normal(N)
            if not dense:
                g *= rng.random(N) < 0.03                   # 3 % non-zero, 10 % kept
            grads.append(g.astype(np.float32))
        _check_step(gpu, ora, grads, f"step {step}", check_state=(step in (3, 6)))
        restaged.append(gpu.topk_stats()[0])
    per_step = np.diff([0] + restaged)
    n_multi = 2 * W
    assert per_step[0] == n_multi                           # nothing to guess from
    assert per_step[1:4].sum() == 0, per_step               # bin 0 guessed and found
    assert per_step[4] == n_multi, per_step                 # the dense step misses
    assert per_step[6] == 0, per_step
    gpu.destroy()


def test_zero_threshold_with_dense_rows_and_kept_zeros():
    """An embedding-like layer: a few rows are dense, the rest exactly zero, and more is kept than is
    non-zero.  Once bin 0 is guessed the first pass lists every non-zero entry; the quarters of
    the dense rows overflow their lists, the first quarters of the layer keep exact zeros (which
    no list holds), and both are taken from Delta quarter by quarter and worker by worker while
    the others are served by the lists.  Every step is exact, payload order included."""
    print("case zero threshold, dense rows", flush=True)
    rows, cols = 96, 672                                    # 8 tiles
    shapes = [(rows, cols, 1), (1, 3 * 8192 + 77, 0)]
    layers = wl.make_layers(shapes)
    N = wl.total_params(layers)
    W = 3
    gpu, ora = H.make_pair(B.ACC_TOPK, layers, W, 10, 1)
    rng = np.random.default_rng(31)
    restaged = []
    for step in range(5):
        grads = []
        for w in range(W):
            g = np.zeros(N, np.float32)
            m = np.zeros((rows, cols), np.float32)
            lo = 88 - 3 * w - (step % 2)                    # six dense rows, elsewhere per worker and step
            m[lo:lo + 6] = rng.standard_normal((6, cols))
            g[:rows * cols] = m.reshape(-1)
            v = rng.standard_normal(N - rows * cols) * (rng.random(N - rows * cols) < 0.02)
            g[rows * cols:] = v
            grads.append(g)
        _check_step(gpu, ora, grads, f"step {step}", check_state=(step in (2, 4)))
        restaged.append(gpu.topk_stats()[0])
    per_step = np.diff([0] + restaged)
    assert per_step[2:].sum() == 0, per_step                # bin 0 guessed and found
    gpu.destroy()


def test_a_sparse_layer_running_dry_is_seen_coming():
    """A sparse gradient (3 % non-zero) whose memory has filled up while little was kept: the first
    step that keeps 10 % again finds more than 10 % non-zero entries (threshold above zero) and
    empties the memory to below that, so from the second step on the threshold is zero.  The step
    that decides the first sees it coming (what it leaves behind plus what a gradient brought in
    when everything non-zero was kept last time is less than k) and guesses bin 0 for the second:
    nothing is staged twice there; every step is exact."""
    print("case sparse layer runs dry", flush=True)
    shapes = [(1, 6 * 8192 + 5, 0), (40, 1031, 1)]
    layers = wl.make_layers(shapes)
    N = wl.total_params(layers)
    W = 2
    gpu, ora = H.make_pair(B.ACC_TOPK, layers, W, 10, 1)
    rng = np.random.default_rng(23)
    restaged = []
    for step in range(12):
        if step in (2, 4, 10):
            # no history: critical (K 10 % stays); stationary norms: K 1 % from step 4; a
            # learning-rate decay: K 10 % again from step 10
            lr_next = 0.01 if step == 10 else 0.1
            ref = ora.detect_regime(0.1, lr_next)
            gpu.detect_regime(0.1, lr_next)
            assert np.array_equal(gpu.get_levels(), ref)
        grads = [(rng.standard_normal(N) * (rng.random(N) < 0.03)).astype(np.float32) for _ in range(W)]
        _check_step(gpu, ora, grads, f"step {step}", check_state=(step in (5, 11)))
        restaged.append(gpu.topk_stats()[0])
    per_step = np.diff([0] + restaged)
    assert list(ora.level) == [1, 1]
    assert per_step[1:4].sum() == 0, per_step               # threshold zero, guessed
    assert per_step[10] == 0, per_step                      # back at K 10 %: more than 10 % non-zero by now
    assert per_step[11] == 0, per_step                      # and dry again, seen coming
    gpu.destroy()



def test_large_tie_classes_take_the_sweeps_and_stay_exact():
    """Quantised values in layers of several tiles: the tie class of the threshold is far larger
    than the per-quarter key lists, for several steps in a row.  While the threshold jumps from
    one quantised value to another the guess misses (the layer is then decided from re-staged
    keys, which is not counted as a tie sweep); once it rests the guess holds, the lists overflow
    and the sweeps take over."""
    print("case tie sweeps", flush=True)
    shapes = [(1, 4 * 8192 + 5, 0), (3, 9000, 1)]
    layers = wl.make_layers(shapes)
    N = wl.total_params(layers)
    gpu, ora = H.make_pair(B.ACC_TOPK, layers, 2, 10, 1)
    rng = np.random.default_rng(9)
    for step in range(9):
        grads = [(rng.integers(-3, 4, N) * 0.25).astype(np.float32) for _ in range(2)]
        _check_step(gpu, ora, grads, f"step {step}", check_state=(step in (1, 3, 8)))
    restaged, swept = gpu.topk_stats()
    assert restaged > 0 and swept > 0, (restaged, swept)
    gpu.destroy()


@pytest.mark.parametrize("n_tiles,k", [(225, 5000), (800, 20000), (3100, 70000)])
def test_more_keys_around_the_threshold_than_the_pick_kernel_holds_in_lds(n_tiles, k):
    """Twelve keys per wave quarter (2048 elements) lie in one level-2 cell of the key space
    (16384 consecutive key values, so with many ties) and the threshold falls among them: every
    quarter's list is complete, but the layer's lists together exceed what the last pick kernel
    gathers in LDS (225 tiles: 10800 keys; 800 tiles: 38400 keys, the larger instantiation of the
    kernel; 3100 tiles: 148800 keys and more quarters than even that one counts in LDS), so it
    works from the lists in device memory.  Second step: no new gradient, the threshold stays in
    the cell with fewer keys left."""
    print(f"case long lists n_tiles={n_tiles} k={k}", flush=True)
    n = n_tiles * 8192
    layers = wl.make_layers([(1, n, 0)])
    gpu, ora = H.make_pair(B.ACC_TOPK, layers, 1, k, k, n)
    rng = np.random.default_rng([21, n_tiles])
    g = rng.random(n).astype(np.float32) * np.float32(0.9)            # all below the cell
    cell = np.uint32(0x3FC00000)                                      # 1.5f: the low 14 key bits are free
    for q in range(4 * n_tiles):
        pos = q * 2048 + rng.choice(2048, 12, replace=False)
        g[pos] = (cell | rng.integers(0, 1 << 14, 12).astype(np.uint32)).view(np.float32)
    g *= rng.choice(np.array([-1.0, 1.0], np.float32), n)
    _check_step(gpu, ora, [g], "step 0", check_state=False)
    _check_step(gpu, ora, [np.zeros(n, np.float32)], "step 1")
    assert gpu.topk_stats()[1] == 0                                   # no list overflowed: no sweeps
    gpu.destroy()


@pytest.mark.parametrize("crit,noncrit", [(99, 60), (100, 51)])
def test_high_keep_ratios_use_the_values_and_holes_layout(crit, noncrit):
    """The paper's own K = 99 % level: layers that keep more than half store values in index
    order plus the indices of the dropped entries.  Batched and call-by-call paths, layers of
    several tiles at misaligned offsets, heavy ties; the decoded payload, the mean, the residual
    and the layout rule itself are compared with the oracle."""
    print(f"case hole layout {crit}/{noncrit}", flush=True)
    shapes = [(1, 3 * 8192 + 77, 0), (37, 1001, 1), (1, 5, 0), (3, 8192, 1), (1, 1, 0), (1, 2, 0)]
    layers = wl.make_layers(shapes)
    N = wl.total_params(layers)
    W = 2
    rng = np.random.default_rng([crit, noncrit])
    for mode in ("all", "calls"):
        gpu, ora = H.make_pair(B.ACC_TOPK, layers, W, crit, noncrit)
        for li, l in enumerate(layers):
            for level, num in ((1, crit), (0, noncrit)):
                fmt, kept, words = B.payload_format(gpu.cfg, li, level)
                k = orc.k_from_fraction(l.numel, num, 100)
                assert kept == k and words == orc.payload_words_packed(l.numel, k)
                assert fmt == (B.ACC_PAYLOAD_VALUES_HOLES if 2 * k > l.numel else B.ACC_PAYLOAD_INDEX_VALUE)
        for step in range(4):
            if step == 2:
                ora.level[:] = 0
                gpu.set_state(H.oracle_state_blob(gpu, ora))
            if step % 2:
                grads = [(rng.integers(-3, 4, N) * 0.25).astype(np.float32) for _ in range(W)]
            else:
                grads = [rng.standard_normal(N).astype(np.float32) for _ in range(W)]
            if mode == "all":
                _check_step(gpu, ora, grads, f"{mode} step {step}", check_state=(step in (1, 3)))
            else:
                out_ref = ora.step(grads)
                dg = [H.to_dev(g) for g in grads]
                out = H.dev_out(N)
                for w in range(W):
                    gpu.compress_step(w, dg[w], 0)
                gpu.aggregate(0)
                gpu.decompress(out)
                H.assert_bits_equal(out.cpu().numpy(), out_ref, f"{mode} step {step}: mean")
                for w in range(W):
                    for li in range(gpu.n_layers):
                        idx, val = gpu.get_payload(w, li)
                        assert np.array_equal(idx, ora.payload[(w, li)][0])
                        H.assert_bits_equal(val, ora.payload[(w, li)][1], "values")
                st = gpu.unpack_state(gpu.get_state())
                H.assert_bits_equal(st["e"], ora.e, f"{mode} step {step}: residual")
        gpu.destroy()


@pytest.mark.parametrize("crit", [10, 99])
def test_support_overlap_matches_the_oracle(crit):
    """Per-layer overlap of the kept coordinates of pairs of workers (Section 4.3), for (index,
    value) payloads (K 10 %) and for values + holes payloads (K 99 %); gradients built as a
    common sparse mean plus dense noise, plus one pure-noise worker."""
    print(f"case overlap K={crit}", flush=True)
    shapes = [(1, 3 * 8192 + 77, 0), (37, 1001, 1), (1, 5, 0), (3, 8192, 1), (1, 1, 0)]
    layers = wl.make_layers(shapes)
    N = wl.total_params(layers)
    W = 3
    gpu, ora = H.make_pair(B.ACC_TOPK, layers, W, crit, 1)
    with pytest.raises(B.AccordionError) as ei:
        gpu.topk_overlap(0, 1)                               # no payloads yet
    assert ei.value.status == B.ACC_ESTATE
    rng = np.random.default_rng(crit)
    mean = np.zeros(N)
    hot = rng.choice(N, N // 10, replace=False)
    mean[hot] = rng.choice([-1.0, 1.0], hot.size) * 5.0
    for step in range(2):
        grads = [(mean + 0.3 * rng.standard_normal(N)).astype(np.float32) for _ in range(2)]
        grads.append(rng.standard_normal(N).astype(np.float32))
        _check_step(gpu, ora, grads, f"step {step}")
        for a, b in ((0, 1), (1, 2), (2, 0), (1, 1)):
            common, kept = gpu.topk_overlap(a, b)
            for li, l in enumerate(layers):
                assert kept[li] == ora.layer_k(li)
                ref = orc.support_overlap(ora.payload[(a, li)][0], ora.payload[(b, li)][0])
                assert common[li] == ref, (step, a, b, li, common[li], ref)
        common, kept = gpu.topk_overlap(0, 1)
        if crit == 10 and step == 0:
            assert common.sum() > 0.9 * kept.sum()           # the paper's "> 90 %" under its model
    with pytest.raises(B.AccordionError):
        gpu.topk_overlap(0, 3)
    gpu.destroy()


def test_call_by_call_equals_step_all_and_is_deterministic():
    layers = wl.make_layers([(20, 900, 1), (1, 64, 0), (9, 9, 1)])
    N = wl.total_params(layers)
    W = 3
    rng = np.random.default_rng(3)
    grads = [[rng.standard_normal(N).astype(np.float32) for _ in range(W)] for _ in range(2)]
    results = []
    for mode in ("all", "calls", "all"):
        gpu, _ = H.make_pair(B.ACC_TOPK, layers, W, 10, 1)
        outs = []
        for step in range(2):
            dg = [H.to_dev(g) for g in grads[step]]
            out = H.dev_out(N)
            if mode == "all":
                gpu.step_all(dg, out)
            else:
                for w in (2, 0, 1):                      # any worker order
                    gpu.compress_step(w, dg[w], 0)
                gpu.aggregate(0)
                gpu.decompress(out)
            outs.append(out.cpu().numpy())
        results.append((outs, gpu.get_state().copy()))
        gpu.destroy()
    for outs, st in results[1:]:
        for a, b in zip(outs, results[0][0]):
            H.assert_bits_equal(a, b, "mean")
        assert np.array_equal(st, results[0][1])


def test_batched_and_call_by_call_steps_interleave():
    """The batched path leaves the residual to the next step's first pass; the call-by-call
    path writes it itself.  Any interleaving of the two, with workers compressed in any order,
    gives the oracle's payloads, means and (read once at the end) memory."""
    print("case mixed paths", flush=True)
    layers = wl.make_layers([(1, 2 * 8192 + 31, 0), (20, 900, 1), (1, 64, 0)])
    N = wl.total_params(layers)
    W = 3
    gpu, ora = H.make_pair(B.ACC_TOPK, layers, W, 10, 1)
    rng = np.random.default_rng(21)
    out = H.dev_out(N)
    for step, mode in enumerate(["all", "calls", "all", "all", "calls", "calls", "all"]):
        if step % 2:
            grads = [(rng.integers(-3, 4, N) * 0.25).astype(np.float32) for _ in range(W)]
        else:
            grads = [rng.standard_normal(N).astype(np.float32) for _ in range(W)]
        if mode == "all":
            _check_step(gpu, ora, grads, f"step {step} {mode}", check_state=False)
            continue
        out_ref = ora.step(grads)
        dg = [H.to_dev(g) for g in grads]
        for w in (1, 2, 0):
            gpu.compress_step(w, dg[w], 0)
        gpu.aggregate(0)
        gpu.decompress(out)
        H.assert_bits_equal(out.cpu().numpy(), out_ref, f"step {step} {mode}: mean")
        for w in range(W):
            for li in range(gpu.n_layers):
                idx, val = gpu.get_payload(w, li)
                assert np.array_equal(idx, ora.payload[(w, li)][0]), f"step {step}: indices"
                H.assert_bits_equal(val, ora.payload[(w, li)][1], f"step {step}: values")
    st = gpu.unpack_state(gpu.get_state())
    H.assert_bits_equal(st["e"], ora.e, "residual at the end")
    H.assert_bits_equal(st["A"], ora.A, "accumulator at the end")
    gpu.flush()                                             # nothing pending any more: a no-op
    assert np.array_equal(gpu.get_state(), gpu.pack_state(st["e"], st["A"], None, st["norm_old"],
                                                          st["has_old"], st["level"]))
    gpu.destroy()


def test_set_state_overrides_a_pending_residual():
    """Importing a state while the residual of the last batched step is still pending must take
    the imported memory as it is (nothing of the old step may be dropped from it)."""
    layers = wl.make_layers([(1, 8192 + 77, 0), (12, 50, 1)])
    N = wl.total_params(layers)
    W = 2
    gpu, ora = H.make_pair(B.ACC_TOPK, layers, W, 10, 1)
    rng = np.random.default_rng(33)
    for step in range(2):                                   # the second step leaves its residual pending
        grads = [rng.standard_normal(N).astype(np.float32) for _ in range(W)]
        _check_step(gpu, ora, grads, f"step {step}", check_state=False)
    ora.e[:] = rng.standard_normal((W, N)).astype(np.float32)   # a memory from elsewhere
    ora.A[:] = 0
    gpu.set_state(H.oracle_state_blob(gpu, ora))
    for step in range(2):
        grads = [rng.standard_normal(N).astype(np.float32) for _ in range(W)]
        _check_step(gpu, ora, grads, f"after import, step {step}", check_state=(step == 1))
    gpu.destroy()


def test_state_machine_errors_come_from_the_host():
    layers = wl.make_layers([(4, 10, 1)])
    gpu, _ = H.make_pair(B.ACC_TOPK, layers, 2, 50, 10)
    g = H.to_dev(np.ones(40, np.float32))
    out = H.dev_out(40)
    with pytest.raises(B.AccordionError) as ei:
        gpu.aggregate(0)
    assert ei.value.status == B.ACC_ESTATE
    with pytest.raises(B.AccordionError):
        gpu.decompress(out)
    gpu.compress_step(0, g, 0)
    with pytest.raises(B.AccordionError) as ei:
        gpu.compress_step(0, g, 0)                       # same worker twice
    assert ei.value.status == B.ACC_ESTATE
    with pytest.raises(B.AccordionError) as ei:
        gpu.compress_step(2, g, 0)                       # worker out of range
    assert ei.value.status == B.ACC_EINVAL
    with pytest.raises(B.AccordionError) as ei:
        gpu.compress_step(1, g, 1)                       # TopK has no phase 1
    assert ei.value.status == B.ACC_EINVAL
    with pytest.raises(B.AccordionError) as ei:
        gpu.detect_regime(0.1, 0.1)                      # inside a step
    assert ei.value.status == B.ACC_ESTATE
    with pytest.raises(B.AccordionError):
        gpu.aggregate(0)                                 # worker 1 missing
    gpu.compress_step(1, g, 0)
    gpu.aggregate(0)
    gpu.decompress(out)
    assert np.all(out.cpu().numpy()[:20] == 1.0)         # k = 20 of 40 equal entries: first 20
    assert np.all(out.cpu().numpy()[20:] == 0.0)
    gpu.destroy()


@pytest.mark.parametrize("pad", [0, 1, 2, 3])
def test_layers_that_start_and_end_anywhere(pad):
    """Every remainder of a layer's size by four, below, at and above the size of a tile, each starting at every
    remainder too (layers that do not start on a 16-byte boundary): the last group of a layer is the only
    partial one.  TopK and the batch-size mode."""
    print(f"case start and end, pad {pad}", flush=True)
    sizes = [pad] * (pad > 0) + [1, 2, 3, 5, 8190, 8191, 8192, 8193, 8195, 2 * 8192 - 1, 2 * 8192 + 2, 3 * 8192 + 3]
    layers = wl.make_layers([(1, n, 0) for n in sizes])
    N, W = wl.total_params(layers), 2
    rng = np.random.default_rng(40 + pad)
    gpu, ora = H.make_pair(B.ACC_TOPK, layers, W, 10, 1)
    bat = B.Accordion(B.ACC_BATCH, H.layer_tuples(layers), W, 1, 1, 100, 0.5, 0, None, batch_multiplier=2)
    out, total = H.dev_out(N), None
    for step in range(4):
        grads = [rng.standard_normal(N).astype(np.float32) for _ in range(W)]
        _check_step(gpu, ora, grads, f"pad {pad} step {step}", check_state=step % 2 == 1)
        bat.step_all([H.to_dev(g) for g in grads], out)
        if step % 2 == 0:
            total = grads
        else:
            sums = [t + g for t, g in zip(total, grads)]
            H.assert_bits_equal(out.cpu().numpy(), (sums[0] + sums[1]) / np.float32(4.0), f"pad {pad} step {step}: batch")
    gpu.destroy()
    bat.destroy()


@pytest.mark.parametrize("case", ["normal", "quantised", "all_equal", "all_zero", "sparse"])
@pytest.mark.parametrize("crit", [1, 10, 99])
def test_single_tile_layers(case, crit):
    """Layers that one workgroup decides from registers: sizes around a wave, a group per thread and the tile, with
    ties that span quarters, exact zeros and almost everything or almost nothing kept."""
    print(f"case single tile {case} K {crit}", flush=True)
    layers = wl.make_layers([(1, n, 0) for n in (1, 4, 63, 65, 255, 1023, 4095, 4097, 8189, 8192)])
    N, W = wl.total_params(layers), 2
    rng = np.random.default_rng(crit)
    gpu, ora = H.make_pair(B.ACC_TOPK, layers, W, crit, 5)
    for step in range(3):
        grads = [_case_values(rng, case, N).astype(np.float32) for _ in range(W)]
        _check_step(gpu, ora, grads, f"{case} K {crit} step {step}", check_state=step == 1)
    gpu.destroy()


@pytest.mark.parametrize("crit", [1, 10])
def test_a_guess_that_starts_inside_a_bin(crit):
    """After enough steps at rest the guess starts a few level-2 cells below the threshold instead of at a whole
    bin.  Then memory and gradients shrink together, by 4 % and by 20 %: the threshold falls below the guess's start,
    inside its bin or just out of it, then far out.  Every step exact, the resting ones without a missed guess."""
    print(f"case guess inside a bin K {crit}", flush=True)
    layers = wl.make_layers([(1, 40 * 8192 + 3, 0), (1, 5, 0), (1, 12 * 8192 + 1, 0)])
    N, W = wl.total_params(layers), 2
    rng = np.random.default_rng(crit)
    gpu, ora = H.make_pair(B.ACC_TOPK, layers, W, crit, 5)
    misses, scale = [], np.float32(1.0)
    for step in range(56):
        if step in (46, 52):
            factor = np.float32(0.96 if step == 46 else 0.8)
            scale *= factor
            ora.e *= factor
            gpu.set_state(H.oracle_state_blob(gpu, ora))
        grads = [rng.standard_normal(N, dtype=np.float32) * scale for _ in range(W)]
        if step < 40:                                        # the checks of the early steps are other tests' work
            ora.step(grads)
            gpu.step_all([H.to_dev(g) for g in grads], H.dev_out(N))
        else:
            _check_step(gpu, ora, grads, f"K {crit} step {step}", check_state=step == 44)
        misses.append(gpu.topk_stats()[0])
    assert misses[45] == misses[30], "missed guesses at rest"
    assert misses[46] > misses[45] and misses[52] > misses[51], "the threshold fell and the guess still held"
    gpu.destroy()


@pytest.mark.parametrize("workers,low", [(1, (0,)), (3, (1,)), (5, (0, 4)), (3, (0, 1, 2))])
def test_lists_too_short_for_some_of_the_workers(workers, low):
    """The lists' floor lies a few cells below the last threshold; the bins are counted from further down.  Memory and gradients
    of some workers shrink by 3 %: their thresholds lie below the floor, in a cell that was counted, and their Delta is read
    instead of the lists, for a minority of the workers beside the others' lists.  Every step exact, payloads included."""
    print(f"case short lists W {workers} low {low}", flush=True)
    layers = wl.make_layers([(1, 9 * 8192 + 3, 0), (1, 5, 0), (23, 1031, 1)])
    N = wl.total_params(layers)
    rng = np.random.default_rng(workers)
    gpu, ora = H.make_pair(B.ACC_TOPK, layers, workers, 10, 5)
    scale = np.ones(workers, np.float32)
    short, restaged = [], []
    for step in range(38):
        if step == 36:
            for w in low:
                scale[w] *= np.float32(0.97)
                ora.e[w] *= np.float32(0.97)
            gpu.set_state(H.oracle_state_blob(gpu, ora))
        grads = [rng.standard_normal(N, dtype=np.float32) * scale[w] for w in range(workers)]
        if step < 35:
            ora.step(grads)
            gpu.step_all([H.to_dev(g) for g in grads], H.dev_out(N))
        else:
            _check_step(gpu, ora, grads, f"W {workers} low {low} step {step}", check_state=step != 36)
        short.append(gpu.topk_short_lists())
        restaged.append(gpu.topk_stats()[0])
    assert short[36] - short[35] >= len(low), "no list was short"
    assert restaged[36] - restaged[35] == short[36] - short[35], "a guess was missed instead"
    gpu.destroy()


@pytest.mark.parametrize("workers,tiles,pad,low,dense", [(5, 30, 0, (1,), (3,)), (7, 30, 3, (0, 6), (2,)), (6, 11, 0, (2, 3), ()), (4, 30, 3, (0, 3), (2,)),
                                                          (32, 650, 0, (0, 7, 31), (8,))])
def test_short_lists_beside_overflowed_ones(workers, tiles, pad, low, dense):
    """Workers `low` have short lists, workers `dense` lists that overflow (all they keep lies in few quarters) and the others
    lists that serve, in one compaction (of a third of the workers at most; beyond, in the fourth case, Delta serves them all); the last case counts with a tile per wave and streams the lists.  Every gradient has exactly
    k entries that are not zero, so the memory is empty after each step and the threshold is the smallest of them: at cell 50 of a
    bin until the run is at rest, then 30 cells lower for `low`, below the floor of the lists (8 cells and at most twice the largest
    recent move, which has faded to 5) but in a bin that was counted."""
    import torch
    print(f"case short beside overflowed W {workers} tiles {tiles} pad {pad}", flush=True)
    n = tiles * 8192 // 10 * 10
    layers = wl.make_layers(([(1, pad, 0)] if pad else []) + [(1, n, 0)])
    N, li, k = wl.total_params(layers), len(layers) - 1, n // 10
    assert workers * tiles < 20000 or N * workers > 64 << 20
    gen = torch.Generator(device="cuda:0")
    gen.manual_seed(workers)
    smallest = lambda cell: 1.0 + (192 + cell) / 512.0
    grads, base = [], []
    for w in range(workers):
        at = torch.arange(k, device="cuda:0") if w in dense else \
            10 * torch.arange(k, device="cuda:0") + torch.randint(10, (k,), generator=gen, device="cuda:0")
        u = torch.rand(k, generator=gen, device="cuda:0")
        u[0] = 0.0
        sign = 1.0 - 2.0 * torch.randint(2, (k,), generator=gen, device="cuda:0")
        g = torch.zeros(N, device="cuda:0")
        if pad:
            g[0] = 1.0
        base.append((at, u, sign))
        grads.append(g)

    def fill(w, cell):
        at, u, sign = base[w]
        s = smallest(cell)
        grads[w][pad + at] = sign * torch.clamp(s * (1.0 + u), min=s)
    for w in range(workers):
        fill(w, 50)
    gpu = B.Accordion(B.ACC_TOPK, H.layer_tuples(layers), workers, 10, 1)
    out = torch.empty(N, device="cuda:0")
    for step in range(28):
        if step == 26:
            for w in low:
                fill(w, 20)
        if step == 25:
            before = gpu.topk_short_lists(), gpu.topk_stats()[0]
        gpu.step_all(grads, out)
        if step < 25:
            continue
        mean = torch.zeros(N, device="cuda:0")
        for g in grads:
            mean += g
        H.assert_bits_equal(out.cpu().numpy(), mean.cpu().numpy() / np.float32(workers), f"step {step}: mean")
        for w in sorted({*low, *dense, workers // 2, workers - 1}):
            idx, val = gpu.get_payload(w, li)
            ref = torch.nonzero(grads[w][pad:])[:, 0]
            assert np.array_equal(idx, ref.cpu().numpy()), f"step {step}: indices of worker {w}"
            H.assert_bits_equal(val, grads[w][pad + ref].cpu().numpy(), f"step {step}: values of worker {w}")
        now = gpu.topk_short_lists(), gpu.topk_stats()[0]
        expected = len(low) if step == 26 else 0
        assert (now[0] - before[0], now[1] - before[1]) == (expected, expected), f"step {step}: short lists, restaged layers"
        before = now
    gpu.destroy()


def test_layers_at_the_edges_of_the_level_2_slot_groups():
    """512 tiles share 32 slots of sixteen tiles, 513 tiles 17 slots of 32, 511 and 497 tiles leave the last slot
    unfilled or with one tile.  A count lost or added twice would miss the guess or move the threshold."""
    print("case slot groups", flush=True)
    sizes = [512 * 8192, 512 * 8192 + 1, 511 * 8192 - 3, 496 * 8192 + 2]
    layers = wl.make_layers([(1, n, 0) for n in sizes])
    N = wl.total_params(layers)
    rng = np.random.default_rng(512)
    gpu, ora = H.make_pair(B.ACC_TOPK, layers, 1, 10, 1)
    batches = [rng.standard_normal(N, dtype=np.float32) for _ in range(2)]
    misses = []
    for step in range(4):
        _check_step(gpu, ora, [batches[step % 2]], f"slot groups step {step}", check_state=step == 3)
        misses.append(gpu.topk_stats()[0])
    assert misses[0] == len(sizes) and misses[3] == misses[0], misses
    gpu.destroy()


@pytest.mark.parametrize("size", [0, 8_400_000])
@pytest.mark.parametrize("pad", [0, 1, 4, 16])
def test_rows_that_a_step_leaves_alone(pad, size):
    """Layers of which a step touches a few rows only, and some not at all: what the first pass does not change it need
    not store, in whole cache lines.  Starts on a 64-byte line, off a 16-byte boundary, on a 16-byte boundary off a line and
    again on a line; rows that end inside a line; negative zeros in the memory and in the gradients; a window end, after
    which the accumulator is written whatever it held.  Memory and accumulator are compared with the oracle bit for bit.  The
    comparison is made in contexts of more than 64 MB of error memory: the layers again in flat buffers of that size, where the third
    worker's memory lies beyond the first 64 MB and is streamed as well."""
    print(f"case untouched rows pad={pad} size={size}", flush=True)
    shapes = ([(1, pad, 0)] if pad else []) + [(300, 84, 1), (1, 12, 0), (200, 100, 1), (6, 50, 1), (40, 672, 1)]
    layers = wl.make_layers(shapes)
    N, W = wl.total_params(layers), 3 if size else 2
    cached = (64 << 20) // 4
    if size:
        assert size % 64 == 0 and size + N < cached <= 2 * size
        gpu, ora = H.make_pair_in(size, B.ACC_TOPK, layers, W, 10, 1)
    else:
        assert N * W < cached
        gpu, ora = H.make_pair(B.ACC_TOPK, layers, W, 10, 1)
    rng = np.random.default_rng([43, pad])
    for step in range(7):
        if step == 3:
            gpu.detect_regime(0.1, 0.1)
            ora.detect_regime(0.1, 0.1)
        if step == 5:                                        # negative zeros where the memory holds zeros
            for w in range(W):
                e = ora.e[w][:N]
                e[(e == 0) & (rng.random(N) < 0.5)] = np.float32(-0.0)
            gpu.set_state(H.oracle_state_blob(gpu, ora))
        grads = []
        for w in range(W):
            g = rng.standard_normal(N)
            for l in layers:
                if l.rows > 1:
                    v = g[l.offset:l.offset + l.numel].reshape(l.rows, l.cols)
                    v *= (rng.random((l.rows, 1)) < (0.0 if step == 4 else 0.06))
                    v[rng.random(l.rows) < 0.1] *= -1.0      # zeros of either sign, but never on top of a negative one
            if step >= 5:
                g = g + 0.0
            grads.append(H.in_buffer(g.astype(np.float32), size or N))
        _check_step(gpu, ora, grads, f"pad {pad} step {step}", check_state=step in (1, 3, 4, 6))
    gpu.destroy()


@pytest.mark.parametrize("crit", [10, 40, 99])
def test_streamed_batched_steps_equal_call_by_call_ones(crit):
    """A context of more than 64 M elements, whose batched steps stream the error memory (beyond 64 MB), the candidate lists
    (K = 10 %) and Delta in the compaction (K = 40 % guesses a band, 99 % has the holes layout), against the call-by-call
    path, which takes every selection from Delta: mean, payloads of the first and last worker, memory, accumulator."""
    print(f"case streamed steps K={crit}", flush=True)
    import torch
    layers = wl.make_layers([(1, 3, 0), (3000, 401, 1), (1, 64, 0), (1200, 768, 1), (1, 8192, 0), (120, 1024, 1)])
    N, W = wl.total_params(layers), 30
    assert N * W > 64 << 20 and 4 * N * W > 224 << 20
    gen = torch.Generator(device="cuda:0")
    results = []
    for mode in ("all", "calls"):
        gpu = B.Accordion(B.ACC_TOPK, H.layer_tuples(layers), W, crit, 1)
        gen.manual_seed(crit)
        out, got = H.dev_out(N), []
        for step in range(4):
            dg = [torch.randn(N, generator=gen, device="cuda:0") for _ in range(W)]
            l = layers[3]
            for g in dg:
                g[l.offset:l.offset + l.numel].view(l.rows, l.cols).mul_(torch.rand(l.rows, 1, generator=gen, device="cuda:0") < 0.06)
            if mode == "all":
                gpu.step_all(dg, out)
            else:
                for w in range(W):
                    gpu.compress_step(w, dg[w], 0)
                gpu.aggregate(0)
                gpu.decompress(out)
            got.append(out.cpu().numpy())
        got += [gpu.get_payload(w, li) for w in (0, W - 1) for li in range(gpu.n_layers)]
        got.append(gpu.get_state().copy())
        results.append(got)
        gpu.destroy()
    for i, (a, b) in enumerate(zip(*results)):
        if isinstance(a, tuple):
            assert np.array_equal(a[0], b[0]) and np.array_equal(H.bits(a[1]), H.bits(b[1])), f"payload {i}"
        else:
            assert np.array_equal(np.ascontiguousarray(a).view(np.uint8), np.ascontiguousarray(b).view(np.uint8)), f"K {crit}: output {i}"


def test_a_tile_per_wave_in_the_counting_kernel():
    """A batched step of more than 20 000 tiles, whose counting kernel takes a tile per wave, against the call-by-call path,
    which takes a quarter per wave: layers of two tiles (the second of one element, of a few, or whole), of one and of three; the first
    step's guess misses everywhere, a layer whose scale jumps misses later, one layer is all ties."""
    print("case wide counting kernel", flush=True)
    import torch
    sizes = [8193, 8192 + 7, 2 * 8192, 5000, 2 * 8192 + 4097]
    layers = wl.make_layers([(1, sizes[i % 5], 0) for i in range(350)])
    N, W = wl.total_params(layers), 32
    assert W * sum(-(-l.numel // 8192) for l in layers) >= 20000
    gen = torch.Generator(device="cuda:0")
    results = []
    for mode in ("all", "calls"):
        gpu = B.Accordion(B.ACC_TOPK, H.layer_tuples(layers), W, 10, 1)
        gen.manual_seed(9)
        out, got = H.dev_out(N), []
        for step in range(4):
            dg = [torch.randn(N, generator=gen, device="cuda:0") for _ in range(W)]
            for g in dg:
                g[layers[0].offset:layers[0].offset + layers[0].numel] *= 64.0 ** step
                g[layers[2].offset:layers[2].offset + layers[2].numel] = 0.5
            if mode == "all":
                gpu.step_all(dg, out)
            else:
                for w in range(W):
                    gpu.compress_step(w, dg[w], 0)
                gpu.aggregate(0)
                gpu.decompress(out)
            got.append(out.cpu().numpy())
        results.append(got + [gpu.get_state().copy()])
        gpu.destroy()
    for i, (a, b) in enumerate(zip(*results)):
        assert np.array_equal(np.ascontiguousarray(a).view(np.uint8), np.ascontiguousarray(b).view(np.uint8)), f"output {i}"


def test_runs_of_tiles_for_one_die():
    """Contexts of more than 1 GiB of error memory take every 256 tiles (half tiles in the compaction) in another order; the
    last 11 of these 1035 keep their own.  32 workers, two steps, against the sorted magnitudes on the device."""
    import torch
    print("case runs of tiles", flush=True)
    W, n = 32, 1035 * 8192 - 5
    layers = wl.make_layers([(1, n, 0)])
    gpu = B.Accordion(B.ACC_TOPK, H.layer_tuples(layers), W, 10, 1)
    k = (n * 10 + 99) // 100
    gen = torch.Generator(device="cuda:0")
    gen.manual_seed(7)
    memory = [torch.zeros(n, device="cuda:0") for _ in range(W)]
    out = torch.empty(n, device="cuda:0")
    for step in range(2):
        grads = [torch.randn(n, generator=gen, device="cuda:0") for _ in range(W)]
        gpu.step_all(grads, out)
        mean = torch.zeros(n, device="cuda:0")
        for w in range(W):
            d = memory[w].add_(grads[w])
            keep = torch.sort(d.view(torch.int32) & 0x7fffffff, descending=True, stable=True).indices[:k]
            mean[keep] += d[keep]
            if w in (0, 17, 31):
                idx, val = gpu.get_payload(w, 0)
                ref = torch.sort(keep).values
                assert np.array_equal(idx, ref.cpu().numpy()), f"step {step}: indices of worker {w}"
                H.assert_bits_equal(val, d[ref].cpu().numpy(), f"step {step}: values of worker {w}")
            d[keep] = 0.0
        H.assert_bits_equal(out.cpu().numpy(), (mean / W).cpu().numpy(), f"step {step}: mean")
    gpu.destroy()
