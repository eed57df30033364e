"""Short attention problems, whose rows are cut into segments over several workgroups: against
the oracle at the edges of the cut, and with workspaces of every size."""
import os
import re

import numpy as np
import pytest

import synth
from parity import O_MAX_ABS, O_MEAN_ABS, compare_outputs, log, to_device

torch = pytest.importorskip("torch")

import paper_2502_20766_amd as fpx


def test_preferred_workspace_covers_the_size_and_is_bounded():
    for seqlens, hq, hkv, d, block in (((1,), 1, 1, 64, 128), ((2048,), 2, 2, 64, 128),
                                       ((4096,), 32, 8, 128, 128), ((300, 1, 4000), 28, 4, 128, 64),
                                       ((6000,), 64, 1, 64, 64), ((131072,), 32, 8, 128, 128)):
        sh = fpx.Shape(np.concatenate([[0], np.cumsum(seqlens)]), hq, hkv, d, block)
        need, best = fpx.attn_workspace_size(sh), fpx.attn_workspace_preferred(sh)
        assert need <= best <= need + (256 << 20)
        if sum(seqlens) > 100000:
            assert best == need


def test_preferred_workspace_fits_the_scratch_array():
    """What fp_sparse_attn_noalloc accepts it runs with the same cuts as fp_sparse_attn: the
    preferred workspace is no larger than the scratch array wherever the required one is not."""
    capped = 0
    for hq, hkv, d in ((32, 32, 128), (32, 8, 128), (28, 4, 128), (64, 64, 64), (16, 16, 128),
                       (8, 1, 64), (40, 40, 128), (1024, 1024, 64)):
        for block in (64, 128):
            for n in (1, 700, 1500, 2049, 3000, 4001, 5900, 8190, 9830, 16384):
                sh = fpx.Shape([0, n], hq, hkv, d, block)
                need, best = fpx.attn_workspace_size(sh), fpx.attn_workspace_preferred(sh)
                if need <= fpx.NOALLOC_SCRATCH_BYTES:
                    assert best <= fpx.NOALLOC_SCRATCH_BYTES, (hq, hkv, d, block, n)
                    capped += best > fpx.NOALLOC_SCRATCH_BYTES - (1 << 20)
    assert capped > 0


def test_no_kernel_waits_for_another_workgroup():
    """A kernel that loops until another workgroup's counter arrives hangs the queue when two
    calls share a workspace against the header's rule (the second call's preparation clears
    the counter): results may be undefined then, an end may not.  No loop of the kernels tests
    a device-scope load, and none sleeps."""
    csrc = os.path.join(os.path.dirname(fpx.__file__), "csrc")
    for name in sorted(os.listdir(csrc)):
        text = re.sub(r"//[^\n]*|/\*.*?\*/", "", open(os.path.join(csrc, name)).read(), flags=re.S)
        assert not re.search(r"\b(while|for)\s*\([^{;]*__hip_atomic_load", text), name
        assert "s_sleep" not in text, name


# seqlens, hq, hkv, d, block, blocks listed per row: lengths around the shortest segment
# (4 blocks) and its multiples, every block, and lists whose ends fall outside the causal range
CASES = [
    ((2048,), 2, 2, 64, 128, "all"),
    ((2048,), 2, 1, 128, 128, "all"),
    ((130, 1, 900, 1152), 6, 3, 128, 128, "edges"),
    ((1500, 65, 700), 8, 2, 128, 64, "edges"),
    ((1000,), 16, 16, 64, 64, "edges"),
    ((4001,), 32, 8, 128, 128, "all"),
    ((1153, 640), 4, 1, 128, 128, "skipped"),
    ((640, 577), 4, 2, 64, 64, "skipped"),
]


@pytest.mark.gpu
@pytest.mark.parametrize("case", CASES, ids=[f"{c[0]}-{c[1]}h{c[2]}-d{c[3]}-b{c[4]}-{c[5]}"
                                             for c in CASES])
def test_split_rows_vs_oracle(case):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    seqlens, hq, hkv, d, block, lists = case
    log(f"[split] {case}")
    kinds = tuple("vs" if h % 2 == 0 else "qa" for h in range(hq))
    spec = synth.LayerSpec("split", seqlens, hq, hkv, d, block, kinds, 8, 0.9, 0.1, 2, 31)
    layer = synth.make_layer(spec)
    rng = np.random.default_rng(17)
    masks, listed = {}, {}
    for s, n in enumerate(seqlens):
        nb = -(-n // block)
        for h in range(hq):
            m = np.tril(np.ones((nb, nb), bool))
            if lists != "all":
                for I in range(nb):
                    want = min(I + 1, int(rng.choice([1, 3, 4, 5, 7, 8, 9, 12, 13])))
                    m[I] = False
                    m[I, rng.choice(I + 1, want, replace=False)] = True
                    m[I, I] = True
            masks[(s, h)] = m
    q, k, v = to_device(layer)
    shape = fpx.Shape(layer.cu_seqlens, hq, hkv, d, block)
    idx = fpx.indices_from_masks(shape, masks, q.device)
    if lists == "skipped":
        # every third row of 5 blocks or more: its first four entries (a whole segment, and
        # the reference of the row's first stages) lie outside the causal range
        nbs = shape.nb()
        tri = np.concatenate([[0], np.cumsum(nbs * (nbs + 1) // 2)])
        off = np.concatenate([[0], np.cumsum(nbs)])
        kb, cnt = idx.kb_idx.cpu().numpy(), idx.kb_cnt.cpu().numpy()
        for (s, h), m in masks.items():
            for I in range(0, int(nbs[s]), 3):
                if cnt[h * off[-1] + off[s] + I] >= 5:
                    at = h * tri[-1] + tri[s] + I * (I + 1) // 2
                    m[I, kb[at:at + 4]] = False
                    kb[at:at + 4] = [-1, I + 1, 8191, I + 7]
        idx.kb_idx.copy_(torch.from_numpy(kb))
    need, best = fpx.attn_workspace_size(shape), fpx.attn_workspace_preferred(shape)
    assert best > need
    outs = []
    for size in (best, best, need, (need + best) // 2, need + 4096):
        ws = torch.full((size,), 0xFF, dtype=torch.uint8, device=q.device)
        o = torch.full_like(q, float("nan"))
        fpx.sparse_attn(q, k, v, idx, out=o, workspace=ws)
        torch.cuda.synchronize()
        outs.append(o.float().cpu().numpy())
        mx, mean = compare_outputs(layer, outs[-1], masks,
                                   rows_per_head=None if sum(seqlens) * hq < 20000 else 6)
        log(f"  workspace {size}: max_abs {mx:.3e} mean_abs {mean:.3e}")
        assert mx <= O_MAX_ABS and mean <= O_MEAN_ABS
    np.testing.assert_array_equal(outs[0], outs[1])
    # another cut of the same rows: float32 merges, then one bf16 rounding each (2^-8 of the
    # value) on top of the two sides' bf16 weights
    for o in outs[2:]:
        assert np.abs(o - outs[0]).max() <= O_MAX_ABS


def _few_long_rows(shape, hq, device):
    """Every fourth row lists every block, the others the first and their own."""
    masks = {}
    for s, nb in enumerate(shape.nb()):
        m = np.tril(np.ones((nb, nb), bool))
        m[np.arange(nb) % 4 != 3] = False
        m[np.arange(nb), 0] = m[np.arange(nb), np.arange(nb)] = True
        for h in range(hq):
            masks[(s, h)] = m
    return masks, fpx.indices_from_masks(shape, masks, device)


@pytest.mark.gpu
@pytest.mark.parametrize("hq,hkv", [(32, 32), (8, 2)])
def test_results_by_workspace(hq, hkv):
    """The fixed scratch array gives the default workspace's bits, also where the array limits
    the cut (32 KV heads); the required workspace cuts no row, so a sequence's output has the
    bits of the sequence alone."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    seqlens, d, block = (2300, 501), 128, 128
    log(f"[split] by workspace, {hq} heads on {hkv}")
    gen = torch.Generator("cuda")
    gen.manual_seed(9)
    q, k, v = (torch.randn(sum(seqlens), h, d, generator=gen, device="cuda").bfloat16()
               for h in (hq, hkv, hkv))
    shape = fpx.Shape([0, 2300, 2801], hq, hkv, d, block)
    masks, idx = _few_long_rows(shape, hq, q.device)
    o = fpx.sparse_attn(q, k, v, idx)
    na = fpx.sparse_attn_noalloc(q, k, v, idx, torch.full_like(q, float("nan")))
    torch.cuda.synchronize()
    assert not bool((o != na).any())

    def uncut(idx, *x):
        ws = torch.empty(fpx.attn_workspace_size(idx.shape), dtype=torch.uint8, device=q.device)
        return fpx.sparse_attn(*x, idx, workspace=ws)

    plain = uncut(idx, q, k, v)
    assert bool((o != plain).any())           # (rows of these lists are cut)
    for s, (t0, t1) in enumerate(((0, 2300), (2300, 2801))):
        alone = fpx.Shape([0, t1 - t0], hq, hkv, d, block)
        ix = fpx.indices_from_masks(alone, {(0, h): masks[(s, h)] for h in range(hq)}, q.device)
        got = uncut(ix, *(x[t0:t1].contiguous() for x in (q, k, v)))
        torch.cuda.synchronize()
        assert not bool((got != plain[t0:t1]).any())


@pytest.mark.gpu
def test_default_workspaces_come_from_the_stream_of_the_call(monkeypatch):
    """A workspace taken from the current stream's memory and used on another stream could still
    be in use there, or be given out again while the call runs."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    gen = torch.Generator("cuda")
    gen.manual_seed(4)
    q, k, v = (torch.randn(1024, 2, 64, generator=gen, device="cuda").bfloat16() for _ in range(3))
    out = fpx.empty_indices(fpx.Shape([0, 1024], 2, 2, 64), q.device)
    o, side = torch.empty_like(q), torch.cuda.Stream()
    ref = fpx.sparse_attn(q, k, v, fpx.select(q, k, [0, 1024], 0.9, 0.1, 1))
    torch.cuda.synchronize()
    seen, empty = [], torch.empty

    def spy(*a, **kw):
        seen.append(torch.cuda.current_stream())
        return empty(*a, **kw)

    monkeypatch.setattr(torch, "empty", spy)

    class Handle:                              # what a caller with a raw handle passes
        cuda_stream = side.cuda_stream

    for stream in (side, Handle()):
        fpx.select(q, k, [0, 1024], 0.9, 0.1, 1, out=out, stream=stream)
        fpx.sparse_attn(q, k, v, out, out=o, stream=stream)
        torch.cuda.synchronize()
        assert len(seen) == 2 and all(s.cuda_stream == side.cuda_stream for s in seen)
        assert torch.cuda.current_stream() == torch.cuda.default_stream()
        assert not bool((o != ref).any())
        seen.clear()
