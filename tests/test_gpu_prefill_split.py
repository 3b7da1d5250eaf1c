"""treewy_chain_prefill at the sizes where its launch changes shape, vs the
float64 oracle, through the C ABI.

A unit is split over four workgroups up to a quarter as many units as CUs
(256), over two up to half, and else resident workgroups walk whole units one
after another; each workgroup's chunk waves and state waves meet at one
barrier per 32-token chunk.  The lengths give one chunk (fp32 tokens), fewer
chunks than chunk waves, one more, and ragged last chunks of 1, 16, 17 and 31
tokens; the unit counts a ragged group of eight (a unit's workgroups are dealt
out in groups of eight units), both edges of each rule, several units per
workgroup, and the sizes that the kernel of one workgroup per unit keeps.  Sampled units are checked; the tolerance is the parity tests'.
"""
import numpy as np
import pytest
import torch

import oracle
from paper_2608_20961_amd import workload as wl
from tests.gpu_harness import DEV, TOL, assert_close, say, warm_state

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def tw():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2608_20961_amd import treewy
    return treewy


CASES = [  # B, H, T, tokens, state
    (1, 1, 33, "bf16", "f32"), (1, 9, 49, "bf16", "bf16"), (1, 64, 96, "bf16", "f32"), (1, 64, 129, "bf16", "bf16"),
    (5, 13, 63, "bf16", "f32"), (2, 64, 145, "bf16", "bf16"), (3, 43, 64, "bf16", "f32"), (4, 64, 65, "bf16", "bf16"),
    (1, 257, 160, "bf16", "f32"), (10, 60, 177, "bf16", "bf16"), (9, 64, 319, "bf16", "f32"), (1, 257, 128, "bf16", "f32"),
    (1, 3, 17, "f32", "f32"), (1, 64, 97, "f32", "f32"), (5, 13, 48, "f32", "f32"), (2, 64, 130, "f32", "f32"),
    (3, 43, 70, "f32", "f32"),
    # ... and the sizes kept by the kernel of one workgroup per unit, in its steady state: three and more chunks of 64 fp32
    # tokens, two to four of 32 bf16 tokens past as many units as CUs
    (3, 43, 200, "f32", "f32"), (1, 257, 321, "f32", "f32"), (3, 43, 129, "f32", "f32"), (1, 257, 97, "bf16", "bf16"),
    (1, 257, 64, "bf16", "f32"), (5, 77, 128, "bf16", "f32"), (5, 77, 33, "bf16", "bf16"),
    # (its three solves, by the last chunk's ancestors: above at most 8 or more than 16, here 9 to 16)
    (3, 43, 81, "f32", "f32"), (5, 77, 49, "bf16", "f32"), (5, 77, 44, "bf16", "bf16"),
]


@pytest.mark.parametrize("B,H,T,dtype,state", CASES)
@pytest.mark.parametrize("in_place", [False, True])
def test_prefill_launch_shapes(tw, B, H, T, dtype, state, in_place):
    w = wl.Workload("prefill", B, H, T, 128, 128, dtype, "chain", T, (1,), (0.85, 0.999), (0.05, 0.95), 16,
                    "chain_depth_0_to_N")
    say("[gpu] prefill %d x %d units, T=%d, %s tokens, %s state, in place %s" % (B, H, T, dtype, state, in_place))
    x = wl.make_inputs(w, seed=31, cfg_key=3100 + T)
    units = wl.sample_units(w, 6)
    S0 = warm_state(w, units, 31, 3101)
    if state == "bf16":
        S0 = wl.round_to_bf16(S0)
    S_all = np.zeros((w.units, 128, 128), dtype=np.float32)
    S_all[units] = S0
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    sdt = torch.bfloat16 if state == "bf16" else torch.float32
    dev = lambda a, d=torch.float32: torch.from_numpy(np.ascontiguousarray(a, dtype=np.float32)).to(DEV).to(d)
    S_d = dev(S_all.reshape(B, H, 128, 128), sdt)
    o = torch.full((B, H, T, 128), float("nan"), dtype=dt, device=DEV)
    S_T = S_d if in_place else torch.full_like(S_d, float("nan"))
    tw.treewy_chain_prefill(S_d, dev(x["q"], dt), dev(x["k"], dt), dev(x["v"], dt), dev(x["alpha"]), dev(x["beta"]),
                            S_T=S_T, o=o)
    torch.cuda.synchronize()
    assert bool(torch.isfinite(o).all()) and bool(torch.isfinite(S_T).all())     # every unit and token was written
    uv = lambda a: a.reshape(w.units, *a.shape[2:])[units]
    S_ref = oracle.chain(S0, uv(x["k"]), uv(x["v"]), uv(x["alpha"]), uv(x["beta"]))
    par = np.tile(np.arange(-1, T - 1, dtype=np.int32), (len(units), 1))
    o_ref, _ = oracle.verify(S0, uv(x["q"]), uv(x["k"]), uv(x["v"]), uv(x["alpha"]), uv(x["beta"]), par)
    assert_close("S_T", S_T.float().cpu().numpy().reshape(w.units, 128, 128)[units], S_ref, TOL[dtype])
    assert_close("o", o.float().cpu().numpy().reshape(w.units, T, 128)[units], o_ref, TOL[dtype])


@pytest.mark.parametrize("dtype,T,H", [("bf16", 49, 385), ("f32", 17, 129), ("f32", 49, 129)])
def test_close_keys(tw, dtype, T, H):
    """A last chunk of 17 tokens with keys close together and gates near one, where what the solve holds in few bits
    shows: 64 units, split by columns, against the same 64 among `H` in the kernel of one workgroup per unit.  Same inputs,
    so the errors against 64 bits compare closely: 1.00 of it at most, and 1.04 to 1.07 with the solve's
    off-diagonal block from pairs of bf16."""
    w = wl.Workload("prefill", 1, H, T, 128, 128, dtype, "chain", T, (1,), (0.9999, 0.9999), (0.9, 1.0), 16, "chain_depth_0_to_N")
    x = wl.make_inputs(w, seed=33, cfg_key=3300)
    rng = np.random.default_rng(33)
    k = rng.standard_normal((1, H, 1, 128)) + 0.3 * rng.standard_normal((1, H, T, 128))
    k = (k / np.linalg.norm(k, axis=-1, keepdims=True)).astype(np.float32)
    x["k"] = wl.round_to_bf16(k) if dtype == "bf16" else k
    S0 = (0.1 * rng.standard_normal((1, H, 128, 128))).astype(np.float32)
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    dev = lambda a, d=torch.float32: torch.from_numpy(np.ascontiguousarray(a, dtype=np.float32)).to(DEV).to(d)
    uv = lambda a: a[0, :64]
    S_ref = oracle.chain(uv(S0), uv(x["k"]), uv(x["v"]), uv(x["alpha"]), uv(x["beta"]))

    def err(n):
        S_T, _ = tw.treewy_chain_prefill(dev(S0[:, :n]), *[dev(x[m][:, :n], dt) for m in ("q", "k", "v")],
                                         *[dev(x[m][:, :n]) for m in ("alpha", "beta")])
        torch.cuda.synchronize()
        return np.linalg.norm(S_T[0, :64].cpu().numpy() - S_ref) / np.linalg.norm(S_ref)

    split, unit = err(64), err(H)
    say("[gpu] close keys, %s tokens, T=%d: error of S_T %.3g split, %.3g whole" % (dtype, T, split, unit))
    assert split <= 1.02 * unit
