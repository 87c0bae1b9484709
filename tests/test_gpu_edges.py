"""Kernel edges on the GPU: row and key counts at the sizes of MFMA blocks (16), halves (32), LDS
tiles (64), waves and work items (256) and one off either side, both head dims, against the oracle
at the bar of the parity tests; and repeated calls at sizes where every tile of a long key stream is
loaded behind the one being computed (a missing wait shows as a difference between calls)."""
import numpy as np
import pytest
import torch

from paper_2606_13872_amd import sra
from sra_inputs import SampleGeom, make_inputs
from test_gpu_parity import check_against_oracle

pytestmark = pytest.mark.gpu

# (gen tokens as 1 x 1 x n, ref frames, ref tokens per frame). At least 16 keys per row: D comes from
# the bf16 O, so dS = P (dP - D) is off by P |O| |dO| 2^-9 whatever its size, and with two keys
# dP - D itself may be that small; over n keys its root mean square is |dO| |V| and |O| falls as
# n^-1/2, which leaves 2^-9 / 4 of it at 16.
EDGES = [(1, 1, 16), (15, 2, 17), (31, 1, 33), (64, 2, 32), (65, 3, 63), (127, 1, 129), (257, 2, 64), (320, 1, 321),
         (383, 1, 385), (513, 2, 255)]


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("gen,frames,ref", EDGES)
def test_edges(gen, frames, ref, d):
    print(f"[edges] gen {gen} ref {frames}x{ref} d {d}", flush=True)
    # a handful of keys leaves outputs of order 1: V and dO at a quarter keep them within the bar
    check_against_oracle([SampleGeom(1, 1, gen, frames, 1, ref)], 2, d, 50 + gen, rms=True,
                         vd_scale=0.25 if gen < 64 else 1.0)


@pytest.mark.parametrize("d,packed", [(64, False), (64, True), (128, False), (128, True)])
def test_long_streams_repeat_bitwise(d, packed):
    samples = [SampleGeom(3, 41, 43, 5, 37, 43, group_frames=2), SampleGeom(2, 40, 40, 0, 1, 1)]
    H = 6
    print(f"[repeat] d {d} packed {packed}", flush=True)
    x = make_inputs(samples, H, d, 60 + d, device="cuda")
    q = {}
    for s in ("gen", "ref"):
        t = [x[f"{n}_{s}"] for n in "qkv"]
        buf = torch.stack(t, dim=1) if packed else None
        q[s] = [buf[:, i] for i in range(3)] if packed else t
    first = None
    for _ in range(6):
        o_gen, o_ref, l_gen, l_ref = sra.forward(*q["gen"], *q["ref"], samples)
        g = sra.backward(*q["gen"], *q["ref"], o_gen, o_ref, l_gen, l_ref, x["do_gen"], x["do_ref"], samples)
        out = {"o_gen": o_gen, "o_ref": o_ref, "l_gen": l_gen, "l_ref": l_ref, **g}
        torch.cuda.synchronize()
        if first is None:
            first = out
            continue
        for n, t in out.items():
            assert torch.equal(t, first[n]), n
    # sum over keys of dV = sum over queries of dO, per head and dim (all rows valid here)
    for h in range(H):
        dv = torch.cat([first["dv_gen"][:, h], first["dv_ref"][:, h]]).double().sum(0)
        do = torch.cat([x["do_gen"][:, h], x["do_ref"][:, h]]).double().sum(0)
        assert float((dv - do).norm() / do.norm()) < 0.04
    assert np.isfinite(float(first["dq_gen"].float().sum()))


@pytest.mark.parametrize("masked", [(0, 500), (130, 700)])
@pytest.mark.parametrize("heads,d", [(3, 128), (1, 64), (24, 64)])
def test_keys_masked_by_an_infinite_head_dim(heads, d, masked):
    """Keys whose first head dim is -inf (the queries' is 1) have scores of -inf: weight 0, also where a
    work item or a piece of a split one begins with them."""
    s = SampleGeom(2, 20, 20, 3, 13, 11)
    print(f"[masked keys] heads {heads} d {d} masked {masked}", flush=True)
    x = make_inputs([s], heads, d, 70, device="cuda")
    x["q_gen"][:, :, 0] = 1
    x["k_gen"][masked[0]:masked[1], :, 0] = float("-inf")
    o, _, lse, _ = sra.forward(*[x[n] for n in ("q_gen", "k_gen", "v_gen", "q_ref", "k_ref", "v_ref")], [s])
    k, v = (torch.cat([x[n + "_gen"], x[n + "_ref"]]).double().cpu() for n in "kv")
    q = x["q_gen"].double().cpu()
    for h in range(heads):
        sc = (q[:, h] @ k[:, h].T) / d ** 0.5
        assert float((lse[h].double().cpu() - torch.logsumexp(sc, -1)).abs().max()) < 1e-3
        want = torch.softmax(sc, -1) @ v[:, h]
        assert float((o[:, h].double().cpu() - want).norm() / want.norm()) < 1e-2  # bf16 P and O: 2.5e-3


@pytest.mark.parametrize("heads,d,split", [(3, 128, True), (1, 64, True), (40, 128, False), (24, 64, False), (80, 128, False),
                                           (80, 64, False)])
def test_rows_masked_by_an_infinite_head_dim(heads, d, split):
    """Rows whose scores are all -inf have LSE = -inf (and O = 0 / 0), in a whole item as in a split one."""
    s = SampleGeom(2, 20, 20, 3, 13, 11)
    assert (sra.launch_info([s], sra.SCHED_FORWARD, heads=heads, head_dim=d)[2] > 0) == split
    print(f"[masked rows] heads {heads} d {d} split {split}", flush=True)
    x = make_inputs([s], heads, d, 71, device="cuda")
    x["q_gen"][:, :, 0] = 1
    for n in ("k_gen", "k_ref"):
        x[n][:, :, 0] = float("-inf")
    o, _, lse, _ = sra.forward(*[x[n] for n in ("q_gen", "k_gen", "v_gen", "q_ref", "k_ref", "v_ref")], [s])
    torch.cuda.synchronize()
    assert bool((lse == float("-inf")).all()) and bool(o.isnan().all())


@pytest.mark.parametrize("heads,d,samples", [
    (16, 64, [SampleGeom(6, 33, 54, 9, 33, 54, group_frames=18)]),  # reference items split, gen items whole
    (16, 128, [SampleGeom(9, 40, 41, 6, 40, 41), SampleGeom(2, 20, 20, 8, 40, 40, group_frames=8)]),  # phases
])
def test_gen_only_calls_are_the_gen_rows_of_the_full_call(heads, d, samples):
    """Bit for bit where heads are pinned to XCDs, too: o, LSE and, for do_ref = 0, dq."""
    print(f"[gen only] heads {heads} d {d}", flush=True)
    x = make_inputs(samples, heads, d, 90, device="cuda")
    x["do_ref"].zero_()
    ins = [x[n] for n in ("q_gen", "k_gen", "v_gen", "q_ref", "k_ref", "v_ref")]
    full = sra.forward(*ins, samples)
    grads = sra.backward(*ins, *full, x["do_gen"], x["do_ref"], samples)
    ins[3] = None
    o, _, lse, _ = sra.forward(*ins, samples, gen_queries_only=True)
    g = sra.backward(*ins, o, None, lse, None, x["do_gen"], None, samples, gen_queries_only=True)
    torch.cuda.synchronize()
    assert torch.equal(o, full[0]) and torch.equal(lse, full[2]) and torch.equal(g["dq_gen"], grads["dq_gen"])
