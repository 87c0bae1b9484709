"""The forward's kernels by items and MFMAs (32x32x16 on 256-row items; 16x16x32 on 256, 384 or 512 rows), at
geometries whose rows and keys end inside a wave, a 16-row block and a key tile, with one token
stride for both streams and with two, and with the mid-span rescale forced: whole heads against
float64, at the bars of the parity tests.

`mid_span_triggers` replays a kernel's key order on the host (each span's full 64-key tiles in span
order, as two 32-key halves) and counts the halves after a wave's first whose overflow check
fires with a finite m, with a sum above 2^17 (a margin over the kernel's 2^16, so that float32
against float64 logits cannot change the count). The lanes that share a query hold, of a half, the
keys 8a + b and 8a + 4 + b (32x32x16: two lanes, 16 keys each) or 4g + b and 16 + 4g + b (16x16x32:
four lanes g, 8 keys each), b < 4.
"""
import math

import numpy as np
import pytest
import torch

from paper_2606_13872_amd import sra
from sra_inputs import SampleGeom, make_inputs

pytestmark = pytest.mark.gpu

BIG, LOG2E = 65536.0, 1.4426950408889634
A, B, C = SampleGeom(1, 30, 30, 4, 31, 33), SampleGeom(1, 25, 31, 5, 23, 29), SampleGeom(1, 25, 31, 3, 23, 29)
# name: (geometry, heads, head dim, MFMA rows, rows of an item, items split, scale that makes the row
# maxima climb)
KERNELS = {
    "mfma32_d64": (B, 80, 64, 32, 256, False, 1.5),
    "mfma32_d64_split": (A, 3, 64, 32, 256, True, 1.5),
    "mfma32_d128": (B, 40, 128, 32, 256, False, 1.0),
    "mfma32_d128_split": (A, 5, 128, 32, 256, True, 1.0),
    "mfma16_256": (A, 40, 128, 16, 256, False, 1.0),
    "mfma16_384": (SampleGeom(1, 32, 33, 5, 25, 31), 80, 128, 16, 384, False, 1.0),
    "mfma16_384_split": (C, 16, 128, 16, 384, True, 1.0),
    "mfma16_512": (SampleGeom(1, 33, 31, 3, 23, 29), 64, 64, 16, 512, False, 1.5),
    "mfma16_512_split": (A, 5, 64, 16, 512, True, 1.5),
}


def _launched(g, heads, d):
    """(MFMA rows, rows of an item, items split) by the launch's items and the rule of the scheduler."""
    n, tile, split = sra.launch_info([g], sra.SCHED_FORWARD, heads=heads, head_dim=d)
    items, spans = sra.launch_export([g], sra.SCHED_FORWARD, heads=heads, head_dim=d)
    steps = sum(int((-(-spans[i[4]:i[4] + i[5], 2] // 64)).sum()) for i in items if i[0] >= 0)
    fills = n > 256 and steps >= 20 * n and steps * 1.5 >= 110 * 256
    return (16 if tile > 256 or (d == 128 and fills) else 32), tile, split > 0


def mid_span_triggers(x, g, scale, mfma, tile):
    """(gen, ref) counts of (wave, half) events in head 0's first two items of each stream."""
    heads, d = x["q_gen"].shape[1:]
    items, spans = sra.launch_export([g], sra.SCHED_FORWARD, heads=heads, head_dim=d)
    q = [x["q_" + s][:, 0].double().cpu().numpy() for s in ("gen", "ref")]
    k = [x["k_" + s][:, 0].double().cpu().numpy() for s in ("gen", "ref")]
    lanes = [[8 * a + 4 * l + b for a in range(4) for b in range(4)] for l in range(2)] if mfma == 32 else \
            [[16 * h + 4 * l + b for h in range(2) for b in range(4)] for l in range(4)]
    rows = 32 if mfma == 32 else tile // 8
    counts = [0, 0]
    for stream in (0, 1):
        for it in items[(items[:, 0] == stream) & (items[:, 1] == 0)][:2]:
            start, length = int(it[2]), int(it[3])
            keys = [k[sp[0]][sp[1]:sp[1] + sp[2] // 64 * 64] for sp in spans[it[4]:it[4] + it[5]]]
            kk = np.concatenate(keys)
            for w in range(0, length, rows):
                s = np.zeros((rows, len(kk)))
                n = min(rows, length - w)
                s[:n] = q[stream][start + w:start + w + n] @ kk.T * (scale * LOG2E)
                m = np.full(rows, -np.inf)
                for h in range(s.shape[1] // 32):
                    b = s[:, 32 * h:32 * h + 32]
                    with np.errstate(over="ignore", invalid="ignore"):
                        sums = np.stack([np.exp2(b[:, l] - m[:, None]).sum(1) for l in lanes])
                    if not np.all(sums <= BIG):
                        counts[stream] += bool(h > 0 and (np.isfinite(m) & (sums > 2 * BIG).any(0)).any())
                        m = np.maximum(m, b.max(1))
    return counts


@pytest.mark.parametrize("strides", [1, 2])
@pytest.mark.parametrize("rescale", [False, True])
@pytest.mark.parametrize("name", list(KERNELS))
def test_whole_heads_match_float64(name, rescale, strides):
    g, heads, d, mfma, tile, split, steep = KERNELS[name]
    assert _launched(g, heads, d) == (mfma, tile, split)
    scale = steep if rescale else 1.0 / math.sqrt(d)
    print(f"[forward tiles] {name} rescale {rescale} strides {strides}", flush=True)
    x = make_inputs([g], heads, d, 80, device="cuda")
    if rescale:
        fires = mid_span_triggers(x, g, scale, mfma, tile)
        assert min(fires) >= 8, fires
    if strides == 2:  # the gen tensors as views of one packed buffer
        buf = torch.stack([x[n + "_gen"] for n in "qkv"], dim=1)
        x.update({n + "_gen": buf[:, i] for i, n in enumerate("qkv")})
    got = sra.forward(*[x[n] for n in ("q_gen", "k_gen", "v_gen", "q_ref", "k_ref", "v_ref")], [g], scale)
    torch.cuda.synchronize()
    frame = g.ref_h * g.ref_w
    for h in (0, heads // 2, heads - 1):
        t = {n: x[n][:, h].double() for n in ("q_gen", "k_gen", "v_gen", "q_ref", "k_ref", "v_ref")}
        k, v = torch.cat([t["k_gen"], t["k_ref"]]), torch.cat([t["v_gen"], t["v_ref"]])
        want = [(t["q_gen"], k, v)]
        want += [tuple(t[n + "_ref"][f * frame:(f + 1) * frame] for n in "qkv") for f in range(g.ref_frames)]
        o, lse = [], []
        for qq, kk, vv in want:
            s = (qq @ kk.T) * scale
            lse.append(torch.logsumexp(s, -1))
            o.append(torch.softmax(s, -1) @ vv)
        for i, (wo, wl) in enumerate(((o[0], lse[0]), (torch.cat(o[1:]), torch.cat(lse[1:])))):
            go, gl = got[i][:, h].double(), got[2 + i][h].double()
            assert float((go - wo).norm() / wo.norm()) <= 1e-2, (h, i)
            assert float((gl - wl).abs().max()) <= 1e-3, (h, i)
            if not rescale:  # a peaked softmax puts |O| near 1, where its bf16 storage alone is 4e-3 off
                assert float((go - wo).abs().max()) <= 1e-2, (h, i)
