"""treewy_snapshot_verify, each wave on rows of its own: every node's state and
output against the float64 oracle, for one node, odd and even counts, the most
nodes, chains (no state read back), trees (states read back) and a tree whose
nodes all hang off the committed state, with fp32 and bf16 tokens; and a bad
parent counts as the committed state."""
import numpy as np
import pytest
import torch

import oracle
from paper_2608_20961_amd import workload as wl
from tests.gpu_harness import TOL, Case, assert_close, say

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def tw():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2608_20961_amd import treewy
    return treewy


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("kind,N", [("chain", 1), ("chain", 2), ("chain", 7), ("tree", 13), ("flat", 5), ("tree", 33),
                                    ("tree", 64), ("bad", 9)])
def test_every_state(tw, kind, N, dtype):
    say("[gpu] snapshot %s N=%d %s" % (kind, N, dtype))
    w = wl.Workload("snap", 2, 3, N, 128, 128, dtype, "chain" if kind == "chain" else "tree", min(N, 6),
                    (N,) if kind != "tree" else (4, 4, 2), (0.85, 0.999), (0.05, 0.95), 16, "uniform_node")
    x = wl.make_inputs(w, seed=5, cfg_key=500 + N)
    if kind == "flat":
        x["parent"][:] = -1
    par_gpu = x["parent"].copy()
    if kind == "bad":
        x["parent"][1, 4], x["parent"][1, 6] = -1, -1
        par_gpu = x["parent"].copy()
        par_gpu[1, 4], par_gpu[1, 6] = 4, -7
    x["path_len"][:] = 0                                 # (no path is committed here)
    case = Case(w, seed=5, inputs=x)
    d = case.device()
    err = torch.zeros(w.B, dtype=torch.int32, device="cuda")
    o, snaps = tw.treewy_snapshot_verify(d["S0"], d["q"], d["k"], d["v"], d["alpha"], d["beta"],
                                         torch.from_numpy(par_gpu).cuda(), err=err)
    torch.cuda.synchronize()
    assert err.tolist() == [0, 1 if kind == "bad" else 0]
    o_ref, _, st_ref, _ = case.oracle(states=True)
    assert_close("o", o.float().cpu().numpy().reshape(w.units, N, 128), o_ref, TOL[dtype])
    # fp32 sums and states: within 1e-5 of the oracle over at most 64 nodes (2^-24 each, 128-term sums)
    assert_close("states", snaps.cpu().numpy().reshape(w.units, N, 128, 128), st_ref, 1e-5)
