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
