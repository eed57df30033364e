"""Selection at the sizes where its launches change: chunk statistics merged by the line pass
(up to 16 chunks of 256 keys), workgroups of 256 threads (up to 16 blocks), Q pooled by the
line pass (up to 10 MB), whole rows of the pooled map in one tile
(up to 128 key blocks), the pattern search in one workgroup (up to 128), line marks made by
the list conversion (up to 8192 tokens), every selection problem in one workgroup (up to
16384 units), against the oracle."""
import pytest

import synth
from parity import (O_MAX_ABS, O_MEAN_ABS, assert_relaxations_bounded, compare_outputs,
                    compare_selection, log, to_device)

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

BASE = synth.SPECS["llama32k"].with_params(hq=4, hkv=2, d=64, head_kinds=("vs", "qa") * 2)

# (seqlens, block, vs_granularity)
CASES = [
    ((8192,), 64, 0),            # 128 blocks, 8192 lines
    ((8193, 700), 64, 0),        # 129 blocks, 8193 lines
    ((11520, 3), 64, 0),         # 180 blocks: 16290 units
    ((11521,), 64, 0),           # 181 blocks: 16471 units
    ((16384, 130), 128, 0),      # 128 blocks, 16384 lines
    ((16385,), 128, 0),          # 129 blocks, 16385 lines
    ((4096, 4097), 128, 0),      # four and five scores per thread, 17 chunks
    ((4096, 1, 300), 128, 0),    # 16 chunks
    ((2048, 5), 128, 0),         # 16 blocks
    ((2049, 129), 128, 0),       # 17 blocks
    ((20480,), 128, 0),          # Q of 10 MB
    ((20481,), 128, 0),          # and one token more
    ((16385, 65), 128, 1),       # block-pooled lines of a long sequence
]


@pytest.mark.parametrize("case", CASES, ids=[f"{c[0]}-b{c[1]}-g{c[2]}" for c in CASES])
def test_selection_at_the_edges_of_its_launches(case):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2502_20766_amd as fpx
    seqlens, block, vsg = case
    log(f"[select edges] {case}")
    spec = BASE.with_seqlens(seqlens, f"edge-{seqlens}-{block}").with_params(block=block)
    layer = synth.make_layer(spec)
    q, k, v = to_device(layer)
    idx = fpx.select(q, k, layer.cu_seqlens, spec.gamma, spec.tau, spec.min_budget, block=block,
                     vs_granularity=vsg)
    o = fpx.sparse_attn(q, k, v, idx)
    torch.cuda.synchronize()
    g = dict(masks=fpx.masks_from_indices(idx), pattern=idx.pattern.cpu().numpy(),
             js=idx.js.cpu().numpy(), units=idx.units.cpu().numpy(), o=o.float().cpu().numpy(),
             idx=idx)
    st = compare_selection(layer, g, spec.gamma, spec.tau, spec.min_budget, vs_granularity=vsg)
    log(f"  {st}")
    assert_relaxations_bounded(st)
    mx, mean = compare_outputs(layer, g["o"], g["masks"], rows_per_head=3)
    assert mx <= O_MAX_ABS and mean <= O_MEAN_ABS


@pytest.mark.parametrize("n", [16384, 16385])
def test_ties_at_the_threshold_take_the_lowest_ids(n):
    """Q = 0 makes every score of a pooled row the same number (1 / (I + 1), in float32 as in
    float64): the cut falls inside a run of equal units, which the lowest ids fill -- with every
    problem in one workgroup, and with the radix passes over slices."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import numpy as np
    import oracle
    import paper_2502_20766_amd as fpx
    log(f"[select ties] {n}")
    spec = BASE.with_seqlens((n,), f"ties-{n}").with_params(hq=2, hkv=1, head_kinds=("vs", "qa"),
                                                            min_budget=1)
    layer = synth.make_layer(spec)
    layer.q[:] = 0.0
    q, k, _ = to_device(layer)
    idx = fpx.select(q, k, layer.cu_seqlens, spec.gamma, spec.tau, spec.min_budget,
                     force_pattern=0)
    masks = fpx.masks_from_indices(idx)
    ref = oracle.select(layer.q, layer.k, layer.cu_seqlens, spec.block, spec.gamma, spec.tau,
                        spec.min_budget, force_pattern=0)
    for h in range(2):
        np.testing.assert_array_equal(masks[(0, h)], ref[0][h]["mask"])


@pytest.mark.parametrize("n", [16384, 16385])
@pytest.mark.parametrize("kind", ["map", "first lines", "late lines"])
def test_ties_over_many_steps_take_the_lowest_ids(kind, n):
    """Runs of equal units that the tie break walks in several steps of 1024, the cut in a late
    one.  Keys outside a window have logit -128, weight 0 in float32; the others logit 0, and
    their number is a power of two, so every score is exact in any order of its sums.
    map: the first 16 key blocks, 1/16 in every longer row (about 1600 of 1800 units taken, over
    6600 ids).  lines: 8192 keys, at the start and at the end: 7373 of the 8192 vertical lines
    and of the slash lines that meet them in every representative row."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import numpy as np
    import oracle
    import paper_2502_20766_amd as fpx
    log(f"[select ties] {kind} {n}")
    spec = BASE.with_seqlens((n,), f"ties-{n}").with_params(hq=2, hkv=1, head_kinds=("vs", "qa"),
                                                            min_budget=1)
    layer = synth.make_layer(spec)
    layer.q[:], layer.k[:] = 0.0, 0.0
    layer.q[..., 0], layer.k[..., 0] = 16.0, -64.0
    last = n - min(spec.block, n)                 # first representative row
    lo, hi = {"map": (0, 2048), "first lines": (0, 8192), "late lines": (last - 8192, last)}[kind]
    layer.k[lo:hi, :, 0] = 0.0
    force = 0 if kind == "map" else 1
    q, k, _ = to_device(layer)
    idx = fpx.select(q, k, layer.cu_seqlens, spec.gamma, spec.tau, spec.min_budget,
                     force_pattern=force)
    masks = fpx.masks_from_indices(idx)
    units = idx.units.cpu().numpy().reshape(2, 2)
    ref = oracle.select(layer.q, layer.k, layer.cu_seqlens, spec.block, spec.gamma, spec.tau,
                        spec.min_budget, force_pattern=force)
    for h in range(2):
        want = ref[0][h]["units"]
        log(f"  units {units[h].tolist()}, oracle {tuple(want)}")
        assert units[h, 0] == want[0] and (kind == "map" or units[h, 1] == want[1])
        assert want[0] > (1600 if kind == "map" else 7000)
        np.testing.assert_array_equal(masks[(0, h)], ref[0][h]["mask"])
