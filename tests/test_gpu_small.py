"""The kernels of few units (drafts of at most 48 nodes, chains of at most 32
tokens, commits), vs the float64 oracle: every wave on its own 16 columns, so
the cases are the node counts around the four-node lane groups and the 16-node
tiles, chains and trees, each type, both sides of the unit count where the
other kernels take over (128 of 256 CUs), ragged groups of eight units, long and bad paths, and
bad parents."""
import numpy as np
import pytest
import torch

import oracle
from paper_2608_20961_amd import workload as wl
from tests.gpu_harness import DEV, TOL, Case, assert_close, say, units_of

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def tw():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2608_20961_amd import treewy
    return treewy


def make(B, H, N, kind, dtype, seed, check=None):
    w = wl.Workload("small", B, H, N, 128, 128, dtype, "chain" if kind == "chain" else "tree",
                    N if kind == "chain" else min(N, 5), (1,) if kind == "chain" else (3,), (0.85, 0.999), (0.05, 0.95), 16,
                    "uniform_node")
    return w, Case(w, seed=seed, inputs=wl.make_inputs(w, seed=seed, cfg_key=800 + N), check_units=check)


@pytest.mark.parametrize("dtype,state", [("bf16", "f32"), ("bf16", "bf16"), ("f32", "f32")])
@pytest.mark.parametrize("B,H,N,kind", [(1, 1, 1, "chain"), (2, 3, 3, "tree"), (1, 9, 4, "chain"), (2, 3, 5, "tree"),
                                        (3, 3, 12, "chain"), (2, 4, 13, "tree"), (5, 13, 16, "chain"), (1, 3, 17, "tree"),
                                        (2, 64, 16, "tree"), (3, 43, 9, "tree"), (6, 64, 15, "tree"), (7, 55, 16, "tree"),
                                        (1, 9, 31, "chain"), (2, 64, 32, "tree"), (2, 3, 33, "tree"), (1, 5, 47, "chain"),
                                        (2, 64, 48, "tree"), (3, 43, 29, "tree"), (3, 43, 48, "tree"), (2, 3, 49, "tree")])
def test_round(tw, B, H, N, kind, dtype, state):
    """verify, commit and the fused call (the committed round's draft again) of one case."""
    say("[gpu] small %d x %d units N=%d %s %s tokens %s state" % (B, H, N, kind, dtype, state))
    w, case = make(B, H, N, kind, dtype, 11, check=wl.sample_units(wl.Workload("s", B, H, N, 128, 128, dtype, "tree", 1, (1,),
                                                                             (0.9, 1), (0, 1), 1, "prefix3"), 6))
    if state == "bf16":
        case.S0 = wl.round_to_bf16(case.S0)
    d = case.device()
    if state == "bf16":
        d["S0"] = d["S0"].to(torch.bfloat16)
    err = torch.zeros(B, dtype=torch.int32, device=DEV)
    ver = [d[n] for n in ("q", "k", "v", "alpha", "beta", "parent")]
    o, U = tw.treewy_verify(d["S0"], *ver, err=err)
    S = tw.treewy_commit(d["S0"], U, d["k"], d["alpha"], d["path"], d["path_len"], parent=d["parent"], err=err)
    S_f, o_f, U_f = tw.treewy_commit_verify(d["S0"], U, d["k"], d["alpha"], d["path"], d["path_len"], *ver,
                                            parent_prev=d["parent"], err=err)
    torch.cuda.synchronize()
    assert int(err.sum()) == 0
    o_ref, U_ref, S_ref = case.oracle()
    tol = TOL[dtype] if state == "f32" else TOL["bf16"]
    assert_close("o", units_of(o, w, case.check), o_ref, tol)
    assert_close("U", units_of(U, w, case.check), U_ref, tol)
    assert_close("S", units_of(S, w, case.check), S_ref, tol)
    assert_close("fused S", units_of(S_f, w, case.check), S_ref, tol)
    c = case.check
    par = np.repeat(case.x["parent"], w.H, axis=0)[c]
    S_in = units_of(S_f, w, c)                           # (verified from the state as written)
    o2, U2 = oracle.verify(S_in, case.unit_view("q"), case.unit_view("k"), case.unit_view("v"), case.unit_view("alpha"),
                           case.unit_view("beta"), par)
    assert_close("fused o", units_of(o_f, w, c), o2, tol)
    assert_close("fused U", units_of(U_f, w, c), U2, tol)


@pytest.mark.parametrize("state", ["f32", "bf16"])
@pytest.mark.parametrize("units,T", [((1, 1), 1), ((2, 3), 4), ((1, 9), 13), ((2, 64), 16), ((3, 43), 16), ((1, 5), 17),
                                     ((2, 3), 31), ((2, 64), 32), ((3, 43), 32)])
def test_prefill(tw, units, T, state):
    B, H = units
    say("[gpu] small prefill %d x %d units T=%d %s state" % (B, H, T, state))
    w, case = make(B, H, T, "chain", "bf16", 12)
    S0 = wl.round_to_bf16(case.S0) if state == "bf16" else case.S0
    d = case.device()
    S0_d = torch.from_numpy(S0.reshape(B, H, 128, 128)).to(DEV).to(torch.bfloat16 if state == "bf16" else torch.float32)
    S_T, o = tw.treewy_chain_prefill(S0_d, d["q"], d["k"], d["v"], d["alpha"], d["beta"])
    in_place = S0_d.clone()
    tw.treewy_chain_prefill(in_place, d["q"], d["k"], d["v"], d["alpha"], d["beta"], S_T=in_place)
    torch.cuda.synchronize()
    assert torch.equal(in_place, S_T)
    args = [case.unit_view(n) for n in ("k", "v", "alpha", "beta")]
    S_ref = oracle.chain(S0, *args)
    o_ref, _ = oracle.verify(S0, case.unit_view("q"), *args, np.tile(np.arange(-1, T - 1, dtype=np.int32), (w.units, 1)))
    assert_close("S_T", units_of(S_T, w, case.check), S_ref, TOL["bf16"])
    assert_close("o", units_of(o, w, case.check), o_ref, TOL["bf16"])


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("L", [0, 1, 3, 4, 5, 7, 8, 9, 16, 23, 24, 25, 40, 41, 56, 57, 63, 64])
def test_commit_path_lengths(tw, L, dtype):
    """Paths of a 64-node chain, read in batches of eight, then sixteen entries, into the commit and the fused call."""
    w, case = make(2, 3, 64, "chain", dtype, 13)
    case.x["path"] = np.tile(np.arange(64, dtype=np.int32), (2, 1))
    case.x["path_len"] = np.full(2, L, dtype=np.int32)
    d = case.device()
    _, U = tw.treewy_verify(d["S0"], *[d[n] for n in ("q", "k", "v", "alpha", "beta", "parent")])
    S = tw.treewy_commit(d["S0"], U, d["k"], d["alpha"], d["path"], d["path_len"])
    now = [d[n][:, :, :5].contiguous() for n in ("q", "k", "v", "alpha", "beta")]
    S_f, _, _ = tw.treewy_commit_verify(d["S0"], U, d["k"], d["alpha"], d["path"], d["path_len"], *now,
                                        d["parent"][:, :5].contiguous(), parent_prev=d["parent"])
    torch.cuda.synchronize()
    _, _, S_ref = case.oracle()
    assert_close("S", units_of(S, w, case.check), S_ref, TOL[dtype])
    assert_close("fused S", units_of(S_f, w, case.check), S_ref, TOL[dtype])
    if L == 0:
        assert torch.equal(S, d["S0"]) and torch.equal(S_f, d["S0"])


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_long_paths_cost_no_more_than_in_one_unit_more(tw, dtype):
    """The fused call of an 8-node draft after a path of 64 entries: half a unit per CU (these kernels) takes no longer
    than one unit more (the others).  Expected 0.82 to 0.89 of it; 1.29 (bf16) and 1.59 (fp32 tokens) were measured when the
    path's entries came a few at a time, so the bound of 1.15 lies well clear of both."""
    half = torch.cuda.get_device_properties(0).multi_processor_count // 2
    g = torch.Generator(device=DEV).manual_seed(1)
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    unit = lambda x: x / x.norm(dim=-1, keepdim=True)

    def graph(B):
        r = lambda *s: torch.randn(*s, generator=g, device=DEV)
        gates = lambda n: 0.9 + 0.09 * torch.rand(B, 1, n, generator=g, device=DEV)
        chain = lambda n: torch.arange(-1, n - 1, dtype=torch.int32, device=DEV).repeat(B, 1).contiguous()
        S, U = 0.1 * r(B, 1, 128, 128), r(B, 1, 64, 128)
        q, k, v = unit(r(B, 1, 8, 128)).to(dt), unit(r(B, 1, 8, 128)).to(dt), r(B, 1, 8, 128).to(dt)
        args = (S, U, unit(r(B, 1, 64, 128)).to(dt), gates(64), chain(64) + 1, torch.full((B,), 64, dtype=torch.int32, device=DEV),
                q, k, v, gates(8), gates(8), chain(8))
        kw = dict(parent_prev=chain(64), S_new=torch.empty_like(S), o=torch.empty_like(v), U=torch.empty(v.shape, device=DEV))
        tw.treewy_commit_verify(*args, **kw)
        torch.cuda.synchronize()
        gr = torch.cuda.CUDAGraph()
        with torch.cuda.graph(gr):
            for _ in range(20):
                tw.treewy_commit_verify(*args, **kw)
        return gr, args, kw                              # (the graph reads and writes these)

    graphs = [graph(half), graph(half + 1)]
    best = [float("inf")] * 2
    for _ in range(20):                                  # in turn
        for i, (gr, _, _) in enumerate(graphs):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            gr.replay()
            b.record()
            torch.cuda.synchronize()
            best[i] = min(best[i], a.elapsed_time(b) * 1e3 / 20)
    say("[gpu] fused, 64 entries, %s tokens: %d units %.2f us, %d units %.2f us" % (dtype, half, best[0], half + 1, best[1]))
    assert best[0] <= 1.15 * best[1], best


@pytest.mark.parametrize("N,H", [(9, 2), (25, 2), (40, 2), (64, 2), (9, 43), (25, 43), (40, 43)])
def test_malformed(tw, N, H):
    """A bad parent counts as -1, a bad path keeps the state, each with its flag and only for its sequence; in 129
    units, and with 64 nodes, by the kernels that these take over from."""
    w, case = make(3, H, N, "chain", "bf16", 14, check=[b * H + h for b in range(3) for h in (0, H - 1)])
    par = case.x["parent"].copy()
    par[1, 4], par[1, 7] = 4, -3
    case.x["parent"][1, 4] = case.x["parent"][1, 7] = -1
    case.x["path_len"][:] = 0
    d = case.device()
    err = torch.zeros(3, dtype=torch.int32, device=DEV)
    o, U = tw.treewy_verify(d["S0"], *[d[n] for n in ("q", "k", "v", "alpha", "beta")], torch.from_numpy(par).to(DEV), err=err)
    torch.cuda.synchronize()
    assert err.tolist() == [0, 1, 0]
    o_ref, U_ref, _ = case.oracle()
    assert_close("o", units_of(o, w, case.check), o_ref, TOL["bf16"])
    assert_close("U", units_of(U, w, case.check), U_ref, TOL["bf16"])
    path = torch.tensor([[0, 1, 2], [0, 2, 1], [0, 1, N]], dtype=torch.int32, device=DEV)
    for plen, flags in (([3, 3, 3], [0, 2, 2]), ([3, 2, 2], [0, 0, 0]), ([4, -1, 0], [2, 2, 0])):
        err.zero_()
        S = tw.treewy_commit(d["S0"], U, d["k"], d["alpha"], path, torch.tensor(plen, dtype=torch.int32, device=DEV), err=err)
        torch.cuda.synchronize()
        assert err.tolist() == flags
        for b in range(3):
            if flags[b]:
                assert torch.equal(S[b], d["S0"][b])


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_tokens_at_element_alignment(tw, dtype):
    """Keys (commit) and all tokens (snapshot baseline) that start in the middle of 16 bytes are taken as before."""
    w, case = make(2, 3, 7, "tree", dtype, 15)
    d = case.device()

    def shifted(t):
        buf = torch.empty(t.numel() + 1, dtype=t.dtype, device=DEV)
        buf[1:] = t.flatten()
        return buf[1:].view(t.shape)

    o, U = tw.treewy_verify(d["S0"], *[d[n] for n in ("q", "k", "v", "alpha", "beta", "parent")])
    k = shifted(d["k"])
    assert k.data_ptr() % 16 and k.is_contiguous()
    S = tw.treewy_commit(d["S0"], U, k, d["alpha"], d["path"], d["path_len"])
    o_s, states = tw.treewy_snapshot_verify(d["S0"], shifted(d["q"]), k, shifted(d["v"]), d["alpha"], d["beta"], d["parent"],
                                            o=shifted(o))
    torch.cuda.synchronize()
    o_ref, _, st_ref, S_ref = case.oracle(states=True)
    assert_close("S", units_of(S, w, case.check), S_ref, TOL[dtype])
    assert_close("o", units_of(o_s, w, case.check), o_ref, TOL[dtype])
    assert_close("states", units_of(states, w, case.check), st_ref, 1e-5)


@pytest.mark.parametrize("state", ["f32", "bf16"])
@pytest.mark.parametrize("N,depth", [(17, 17), (32, 8), (48, 8), (48, 48), (40, 4)])
def test_close_keys(tw, N, depth, state):
    """Keys close together and gates near one: the solve cancels most of R, so what it holds in few bits shows in U.  The
    same draft in 129 units runs verify.hip; the error against 64 bits may be no more than a fifth above its, which
    other random inputs need (measured 0.2 to 1.09 of it; with the off-diagonal products in pairs of bf16 it was 1.28 to 1.6)."""
    def err(B, H):
        w = wl.Workload("close", B, H, N, 128, 128, "bf16", "chain" if depth == N else "tree", depth,
                        (1,) if depth == N else (3,), (0.9999, 0.9999), (0.9, 1.0), 16, "uniform_node")
        x = wl.make_inputs(w, seed=16, cfg_key=816)
        rng = np.random.default_rng(16)
        k = rng.standard_normal((B, H, 1, 128)) + 0.1 * rng.standard_normal((B, H, N, 128))
        x["k"] = wl.round_to_bf16((k / np.linalg.norm(k, axis=-1, keepdims=True)).astype(np.float32))
        case = Case(w, seed=16, cfg_key=816, inputs=x, check_units=wl.sample_units(w, 24))
        if state == "bf16":
            case.S0 = wl.round_to_bf16(case.S0)
        d = case.device()
        S0 = d["S0"].to(torch.bfloat16) if state == "bf16" else d["S0"]
        _, U = tw.treewy_verify(S0, *[d[n] for n in ("q", "k", "v", "alpha", "beta", "parent")])
        torch.cuda.synchronize()
        _, U_ref, _ = case.oracle()
        return np.linalg.norm(units_of(U, w, case.check) - U_ref) / np.linalg.norm(U_ref)

    here, there = err(3, 8), err(3, 43)
    say("[gpu] close keys N=%d depth %d, %s state: error of U %.3g in 24 units, %.3g in 129" % (N, depth, state, here, there))
    assert here <= 1.2 * there
