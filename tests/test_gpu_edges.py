"""GPU parity at the sizes and values where a kernel or a rule of its dispatch can go wrong, against the CPU
oracle."""
import ctypes

import numpy as np
import pytest

import paper_2502_20704_amd as fsd
from paper_2502_20704_amd import synth
from tests import parity_util as pu
from tests.test_gpu_parity import (_random_tree_inputs, check_rfsd, check_sd, check_sd_tree, check_warped, run_chain,
                                   run_rfsd, run_sd_tree, run_tree, run_warped)

pytestmark = pytest.mark.gpu
both_routes = pytest.mark.usefixtures("route")   # see conftest.py


@pytest.fixture(scope="module")
def torch_cuda():
    import torch

    assert torch.cuda.is_available(), "these tests need the MI355X"
    fsd.library()
    return torch


@pytest.mark.parametrize("V", [5, 2047, 33001, 131072, 140008])
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_selection_by_value(torch_cuda, oracle, V, dtype):
    """The cut of the warpers where the bins of the value histogram end: rows wider than its range, rows
    that temperature has made narrower than a bin, masked entries (-inf, and the lowest finite value), a
    crossing in the last bin, a row of two values, rows that are not 16-byte aligned or longer than what
    the kernel keeps in registers.  The cut is exact wherever the nucleus mass is not within 1e-5 of top-p."""
    rng = np.random.default_rng(V)
    B, K = 6, 1
    t = (rng.standard_normal((B, K + 1, V)) * 3).astype(np.float32)
    t[1, :, 2:] -= np.float32(60.0)                                   # two entries far above all others
    t[2, :, rng.permutation(V)[: V // 2]] = -np.inf                   # half of the row masked
    t[3, :, rng.permutation(V)[: V // 2]] = np.float32(-3.0e38)       # masked with a finite value
    t[4] = np.where(rng.random((K + 1, V)) < 0.5, 1.0, -1.0)          # two values
    t[5] *= np.float32(1e-3)                                          # nearly flat
    d = (t[:, :K] + rng.standard_normal((B, K, V)).astype(np.float32) * 0.5).astype(np.float32)
    cand = rng.integers(0, V, (B, K)).astype(np.int32)
    inp = dict(target=t, draft=d, cand=cand)
    if dtype == "bf16":
        inp = dict(target=synth.to_bf16_bits(t), draft=synth.to_bf16_bits(d), cand=cand)
    for kw in (dict(top_p=0.4), dict(top_p=0.999), dict(top_k=3), dict(top_k=600), dict(top_k=max(1, V - 2)),
               dict(temperature=900.0, top_p=0.7), dict(temperature=2.0 ** -9, top_k=700, top_p=0.9)):
        print("selection by value", V, dtype, kw, flush=True)
        g = run_warped(torch_cuda, inp, 0.1, fsd.DIV_TV, fsd.SAMPLE, 9, 4, **kw)
        o = oracle.verify_chain_warped(inp["target"], inp["draft"], inp["cand"], 0.1, fsd.DIV_TV, fsd.SAMPLE, 9, 4, **kw)
        active = 0 < kw.get("top_k", 0) < V or kw.get("top_p", 1.0) < 1.0
        check_warped(g, o, 0.1, pu.rel_tol(dtype), f"selection by value V={V} {dtype} {kw}", cut_active=active,
                     envelope=pu.Envelope(dtype))


# entries a team member holds: 3072 (bfloat16 JS, TV), 2048 (the other kernels); a slot: 8 or 4
@both_routes
@pytest.mark.parametrize("V", [3, 7, 8, 9, 15, 2047, 2049, 3071, 3073, 6151])
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_ragged_rows(torch_cuda, oracle, V, dtype):
    """Rows that are not 16-byte aligned, through every entry point: rows shorter than a slot, rows whose last slot
    is all that the team's last member has, and rows one entry short of or past a member's share.  The last row of
    each tensor ends its allocation's used part, so its last slot is the one that must not reach behind."""
    inp = synth.chain_inputs(3, 4, V, dtype, "gauss2", 1.0, seed=V)
    tol, env = pu.rel_tol(dtype), pu.Envelope(dtype)
    for div in (fsd.DIV_JS, fsd.DIV_TV, fsd.DIV_KL):
        for mode in (fsd.SAMPLE, fsd.GREEDY):
            print("ragged", V, dtype, div, mode, flush=True)
            g = run_chain(torch_cuda, inp, 0.1, div, mode, seed=5, offset=2)
            o = oracle.verify_chain(inp["target"], inp["draft"], inp["cand"], 0.1, div, mode, seed=5, offset=2)
            pu.check_chain(g, o, 0.1, tol, f"ragged V={V} {dtype} div={div}", envelope=env)
    g = run_rfsd(torch_cuda, inp, 0.1, fsd.DIV_JS, seed=5, offset=2)
    o = oracle.rfsd_verify_chain(inp["target"], inp["draft"], inp["cand"], 0.1, fsd.DIV_JS, seed=5, offset=2)
    check_rfsd(g, o, 0.1, tol, f"ragged rFSD V={V} {dtype}", envelope=env)
    d = pu.to_dev(inp, ("target", "draft", "cand"))
    out = fsd.sd_verify_chain(d["target"], d["draft"], d["cand"], seed=5, offset=2)
    torch_cuda.cuda.synchronize()
    o = oracle.sd_verify_chain(inp["target"], inp["draft"], inp["cand"], seed=5, offset=2)
    check_sd(pu.host(out, pu.SD_KEYS), o, f"ragged SD V={V} {dtype}")
    tin = _random_tree_inputs(np.random.default_rng(V), 3, 9, V, dtype)
    g = run_tree(torch_cuda, tin, 0.1, fsd.DIV_JS, 9, seed=5, offset=2)
    o = oracle.verify_tree(tin["target"], tin["draft"], tin["node_tokens"], tin["parent"], 9, 0.1, fsd.DIV_JS, seed=5, offset=2)
    pu.check_tree(g, o, 0.1, tol, f"ragged tree V={V} {dtype}", envelope=env)
    g = run_sd_tree(torch_cuda, tin, 9, fsd.SAMPLE, seed=5, offset=2)
    o = oracle.sd_verify_tree(tin["target"], tin["draft"], tin["node_tokens"], tin["parent"], 9, fsd.SAMPLE, seed=5, offset=2)
    check_sd_tree(g, o, f"ragged SD tree V={V} {dtype}", tin)


@both_routes
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_rows_on_odd_addresses(torch_cuda, oracle, dtype):
    """Tensors whose first row starts one element past a 16-byte boundary (V a multiple of the slot)."""
    B, K, V = 2, 3, 4096
    inp = synth.chain_inputs(B, K, V, dtype, "peaked", 1.0, seed=3)
    d = pu.to_dev(inp, ("target", "draft", "cand"))

    def shifted(t):
        buf = torch_cuda.empty(t.numel() + 1, dtype=t.dtype, device="cuda")
        buf[1:] = t.reshape(-1)
        return buf[1:].view(t.shape)

    for div in (fsd.DIV_JS, fsd.DIV_KL):
        out = fsd.fsd_verify_chain(shifted(d["target"]), shifted(d["draft"]), d["cand"], 0.1, div, seed=5, offset=2)
        torch_cuda.cuda.synchronize()
        o = oracle.verify_chain(inp["target"], inp["draft"], inp["cand"], 0.1, div, seed=5, offset=2)
        pu.check_chain(pu.host(out, pu.CHAIN_KEYS), o, 0.1, pu.rel_tol(dtype), f"odd addresses {dtype} div={div}",
                       envelope=pu.Envelope(dtype))


@both_routes
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_every_call_on_odd_addresses(torch_cuda, oracle, dtype):
    """The entry points beside the plain chain call, on tensors whose first row starts one element past a 16-byte
    boundary (V a multiple of the slot)."""
    def shifted(d, *names):
        out = dict(d)
        for name in names:
            buf = torch_cuda.empty(d[name].numel() + 1, dtype=d[name].dtype, device="cuda")
            buf[1:] = d[name].reshape(-1)
            out[name] = buf[1:].view(d[name].shape)
        return out

    V, tol, env = 4096, pu.rel_tol(dtype), pu.Envelope(dtype)
    inp = synth.chain_inputs(3, 4, V, dtype, "gauss2", 1.0, seed=8)
    d = shifted(pu.to_dev(inp, ("target", "draft", "cand")), "target", "draft")
    print("odd addresses", dtype, "sd", flush=True)
    out = fsd.sd_verify_chain(d["target"], d["draft"], d["cand"], seed=5, offset=2)
    torch_cuda.cuda.synchronize()
    check_sd(pu.host(out, pu.SD_KEYS), oracle.sd_verify_chain(inp["target"], inp["draft"], inp["cand"], seed=5, offset=2),
             f"odd addresses SD {dtype}")
    print("odd addresses", dtype, "rfsd", flush=True)
    out = fsd.rfsd_verify_chain(d["target"], d["draft"], d["cand"], 0.1, fsd.DIV_JS, seed=5, offset=2)
    torch_cuda.cuda.synchronize()
    check_rfsd(pu.host(out, pu.RFSD_KEYS), oracle.rfsd_verify_chain(inp["target"], inp["draft"], inp["cand"], 0.1, fsd.DIV_JS, seed=5, offset=2),
               0.1, tol, f"odd addresses rFSD {dtype}", envelope=env)
    for kw in (dict(top_k=40, top_p=0.9), dict(top_p=0.8)):
        print("odd addresses", dtype, kw, flush=True)
        out = fsd.fsd_verify_chain_warped(d["target"], d["draft"], d["cand"], 0.1, fsd.DIV_TV, fsd.SAMPLE, 5, 2, **kw)
        torch_cuda.cuda.synchronize()
        g = pu.host(out, pu.CHAIN_KEYS)
        g["threshold"] = fsd.debug_warp_thresholds(out, 3, 4, V, fsd.BF16 if dtype == "bf16" else fsd.F32).cpu().numpy()
        o = oracle.verify_chain_warped(inp["target"], inp["draft"], inp["cand"], 0.1, fsd.DIV_TV, fsd.SAMPLE, 5, 2, **kw)
        check_warped(g, o, 0.1, tol, f"odd addresses warped {dtype} {kw}", envelope=env)
    tin = _random_tree_inputs(np.random.default_rng(8), 3, 9, V, dtype)
    t = shifted(pu.to_dev(tin, ("target", "draft", "node_tokens", "parent")), "target", "draft")
    print("odd addresses", dtype, "trees", flush=True)
    out = fsd.fsd_verify_tree(t["target"], t["draft"], t["node_tokens"], t["parent"], 9, 0.1, fsd.DIV_JS, seed=5, offset=2)
    torch_cuda.cuda.synchronize()
    o = oracle.verify_tree(tin["target"], tin["draft"], tin["node_tokens"], tin["parent"], 9, 0.1, fsd.DIV_JS, seed=5, offset=2)
    pu.check_tree(pu.host(out, pu.TREE_KEYS), o, 0.1, tol, f"odd addresses tree {dtype}", envelope=env)
    out = fsd.sd_verify_tree(t["target"], t["draft"], t["node_tokens"], t["parent"], 9, fsd.SAMPLE, seed=5, offset=2)
    torch_cuda.cuda.synchronize()
    o = oracle.sd_verify_tree(tin["target"], tin["draft"], tin["node_tokens"], tin["parent"], 9, fsd.SAMPLE, seed=5, offset=2)
    check_sd_tree(pu.host(out, pu.TREESD_KEYS), o, f"odd addresses SD tree {dtype}", tin)


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("mode", [fsd.SAMPLE, fsd.GREEDY])
def test_residual_without_a_positive_part(torch_cuda, oracle, dtype, mode):
    """Strict SD rejects a token whose draft probability is a little larger than its target probability, both so
    small (e^-30) that the other entries' p - q vanish in binary32: no entry of the residual has any mass and the
    token comes from the target row itself, which is what FSD draws when it rejects (same random stream)."""
    B, V = 64, 4099
    rng = np.random.default_rng(7)
    t = (rng.standard_normal((B, 2, V)) * 2).astype(np.float32)
    t[:, 0, 11] = -30.0
    d = t[:, :1].copy()
    d[:, 0, 11] = -29.0                    # accepted with probability e^-1
    cand = np.full((B, 1), 11, dtype=np.int32)
    if dtype == "bf16":
        t, d = synth.to_bf16_bits(t), synth.to_bf16_bits(d)
    inp = dict(target=t, draft=d, cand=cand)
    dv = pu.to_dev(inp, ("target", "draft", "cand"))
    plain = fsd.fsd_verify_chain(dv["target"], dv["draft"], dv["cand"], -1.0, fsd.DIV_TV, mode, seed=6, offset=3)
    for call in (lambda: fsd.sd_verify_chain(dv["target"], dv["draft"], dv["cand"], mode, seed=6, offset=3),
                 lambda: fsd.rfsd_verify_chain(dv["target"], dv["draft"], dv["cand"], -1.0, fsd.DIV_TV, mode, seed=6, offset=3)):
        out = call()
        torch_cuda.cuda.synchronize()
        n, tok = out["accept_len"].cpu().numpy(), out["out_tokens"].cpu().numpy()
        o = oracle.sd_verify_chain(inp["target"], inp["draft"], inp["cand"], mode, seed=6, offset=3)
        assert (n == o["accept_len"]).all() and (out["row_status"].cpu().numpy() == 0).all()
        rejected = n == 0
        assert 20 <= rejected.sum() <= 60
        assert (tok[rejected, 0] == plain["out_tokens"].cpu().numpy()[rejected, 0]).all()


# a wavefront's lanes hold 64 children; a workgroup keeps 3072 slots of a bfloat16 row, 4096 of a binary32 one (8
# workgroups a tree; 256 compute units hold 5 a tree for 44 trees)
@pytest.mark.parametrize("B,N,V,dtype", [(3, 64, 300, "bf16"), (3, 65, 300, "f32"), (2, 130, 77, "bf16"), (2, 5, 150000, "bf16"),
                                         (2, 5, 200001, "bf16"), (2, 5, 200004, "f32"), (40, 6, 20000, "f32"),
                                         (2, 5, 131072, "f32"), (2, 5, 131073, "f32"), (2, 5, 131076, "f32"), (44, 3, 128256, "bf16")])
def test_sd_tree_walk_edges(torch_cuda, oracle, B, N, V, dtype):
    """Strict SD over star-shaped trees (every rejection is followed by another sibling): more children than a
    wavefront has lanes, and rows around what the walk keeps in registers."""
    inp = _random_tree_inputs(np.random.default_rng(N + V), B, N, V, dtype, star=True, noise=(1.5, 3.0))
    g = run_sd_tree(torch_cuda, inp, 1, fsd.SAMPLE, seed=3, offset=1)
    o = oracle.sd_verify_tree(inp["target"], inp["draft"], inp["node_tokens"], inp["parent"], 1, fsd.SAMPLE, seed=3, offset=1)
    r = check_sd_tree(g, o, f"walk edges B={B} N={N} V={V} {dtype}", inp)
    print(r, "tried", (~np.isnan(o["log_ratio"])).sum(1), flush=True)


# (a workgroup's share of the last two rows is more than the walk keeps of a row)
@pytest.mark.parametrize("V,dtype", [(4100, "bf16"), (4100, "f32"), (4101, "bf16"), (200001, "bf16"), (200004, "f32")])
@pytest.mark.parametrize("where", ["draft", "target", "both"])
@pytest.mark.parametrize("value", [-np.inf, -3.3e38])
def test_sd_tree_masked_rows(torch_cuda, oracle, V, dtype, where, value):
    """Strict SD over trees whose rows are cut to a few entries, by -inf or by a finite value far below the others:
    a masked entry has probability 0, so where the draft alone is cut the target's mass there stays in the
    distribution after a rejection.  Stars, in which every rejection but the last is followed by a sibling."""
    rng = np.random.default_rng(V)
    B, N = (2, 5) if V > 100000 else (8, 8)
    t = (rng.standard_normal((B, N + 1, V), dtype=np.float32) * np.float32(2))
    d = t[:, :1] + rng.standard_normal((B, N, V), dtype=np.float32) * np.float32(2.5)
    if where != "draft":
        t[:, :, rng.permutation(V)[: V // 2]] = value
    if where != "target":
        low = np.partition(d, V - V // 8, axis=2)[:, :, V - V // 8, None]
        d[d < low] = value
    q = np.exp(d.astype(np.float64) - d.max(axis=2, keepdims=True))
    toks = np.array([[rng.choice(V, p=q[b, j] / q[b, j].sum()) for j in range(N)] for b in range(B)], dtype=np.int32)
    if dtype == "bf16":
        t, d = synth.to_bf16_bits(t), synth.to_bf16_bits(d)
    inp = dict(target=t, draft=d, node_tokens=toks, parent=np.full((B, N), -1, dtype=np.int32))
    g = run_sd_tree(torch_cuda, inp, 1, fsd.SAMPLE, seed=3, offset=1)
    o = oracle.sd_verify_tree(inp["target"], inp["draft"], inp["node_tokens"], inp["parent"], 1, fsd.SAMPLE, seed=3, offset=1)
    tried = (~np.isnan(o["log_ratio"])).sum(1)
    print("masked rows", V, dtype, where, value, "tried", tried, flush=True)
    assert tried.max() >= 3
    check_sd_tree(g, o, f"masked rows V={V} {dtype} {where} {value}", inp)


@pytest.mark.parametrize("star", [False, True])
@pytest.mark.parametrize("V,dtype", [(2048, "bf16"), (4100, "bf16"), (128256, "bf16"), (2050, "f32"), (40004, "f32")])
def test_sd_tree_siblings_share_sums(torch_cuda, oracle, V, dtype, star):
    """Strict SD over trees: siblings share their target row's sum instead of forming it again.  A star (one row for
    all), random trees (runs of siblings of any length, the teams' runs of pairs crossing sequences), and an
    unusable shared row, which must spoil every pair that refers to it and no other sequence."""
    B, N = (3, 7) if V > 100000 else (5, 24)
    inp = _random_tree_inputs(np.random.default_rng(V), B, N, V, dtype, star=star)
    depth = 1 if star else N
    g = run_sd_tree(torch_cuda, inp, depth, fsd.SAMPLE, seed=3, offset=1)
    o = oracle.sd_verify_tree(inp["target"], inp["draft"], inp["node_tokens"], inp["parent"], depth, fsd.SAMPLE, seed=3, offset=1)
    check_sd_tree(g, o, f"siblings share sums V={V} {dtype} star={star}", inp)
    inp["target"][1, 0, V // 2] = np.uint16(0x7FC0) if dtype == "bf16" else np.float32(np.nan)
    g = run_sd_tree(torch_cuda, inp, depth, fsd.SAMPLE, seed=3, offset=1)
    assert g["row_status"][1] == fsd.ROW_NONFINITE and (np.delete(g["row_status"], 1) == 0).all()
    assert (g["path_nodes"][1] == -1).all() and (g["out_tokens"][1] == -1).all()


# W: workgroups a row where the setting allows them, under top-k and under top-p alone.  A split selection takes rows of
# a length that depends on the setting, the type and the alignment, 16 KB of exchange words a sequence (K times the
# row's wavefronts: 256), at most a workgroup per 1024 slots and per unit of 256 / B, and at most 5120 slots a workgroup.
@pytest.mark.parametrize("B,K,V,dtype,W", [
    (2, 5, 8200, "bf16", (1, 1)), (3, 5, 40000, "bf16", (1, 1)), (3, 5, 16004, "f32", (1, 1)), (300, 2, 9001, "bf16", (1, 1)),
    (2, 25, 20000, "bf16", (1, 1)),                                                   # (all of these: too little room)
    (2, 64, 8192, "bf16", (1, 1)), (2, 64, 8200, "bf16", (1, 2)), (2, 32, 15999, "bf16", (1, 1)), (2, 32, 16001, "bf16", (1, 2)),
    (2, 26, 23992, "bf16", (1, 3)), (2, 22, 24000, "bf16", (3, 3)), (2, 22, 23999, "bf16", (1, 3)), (2, 22, 24001, "bf16", (3, 3)),
    (2, 16, 32000, "bf16", (4, 4)), (2, 13, 40003, "bf16", (5, 5)), (2, 11, 48000, "bf16", (6, 6)), (2, 10, 57000, "bf16", (7, 7)),
    (2, 9, 131073, "bf16", (8, 8)), (2, 5, 327680, "bf16", (8, 8)), (2, 5, 327688, "bf16", (1, 1)),
    (2, 32, 15999, "f32", (1, 1)), (2, 32, 16001, "f32", (1, 4)), (2, 26, 19996, "f32", (1, 1)), (2, 26, 20000, "f32", (1, 5)),
    (2, 26, 19999, "f32", (1, 5)), (2, 26, 20001, "f32", (5, 5)), (2, 13, 39996, "f32", (1, 8)), (2, 13, 40000, "f32", (8, 8)),
    (2, 9, 163840, "f32", (8, 8)), (2, 9, 163844, "f32", (1, 1)),
    (88, 22, 24000, "bf16", (2, 2)), (129, 22, 24000, "bf16", (1, 1))])
def test_selection_by_several_workgroups(torch_cuda, oracle, B, K, V, dtype, W):
    """The warpers' cut where several workgroups share a row: both sides of every line of the rule that splits a
    row, every number of workgroups, unaligned rows, lists that overflow (equal entries, masked rows), and a graph's
    worth of repeats on one workspace (the counters and words of the last call must not matter)."""
    rng = np.random.default_rng(V + B)
    t = (rng.standard_normal((B, K + 1, V), dtype=np.float32) * np.float32(3))
    t[0] = np.float32(0.5)                                             # all equal: every list overflows
    t[1, :, rng.permutation(V)[: V - 700]] = -np.inf                   # fewer entries than threads
    d = (t[:, :K] + rng.standard_normal((B, K, V), dtype=np.float32) * np.float32(0.3))
    cand = rng.integers(0, V, (B, K)).astype(np.int32)
    inp = dict(target=t, draft=d, cand=cand)
    if dtype == "bf16":
        inp = dict(target=synth.to_bf16_bits(t), draft=synth.to_bf16_bits(d), cand=cand)
    dev = pu.to_dev(inp, ("target", "draft", "cand"))
    code = fsd.BF16 if dtype == "bf16" else fsd.F32
    ws = torch_cuda.empty(fsd.fsd_workspace_bytes(B, K, V, code) + 256, dtype=torch_cuda.uint8, device="cuda")
    ws.random_(0, 256)
    for kw in (dict(top_k=40, top_p=0.9), dict(top_p=0.8), dict(top_k=512), dict(temperature=0.5, top_p=0.99))[:2 if B > 80 else 4]:
        print("split selection", B, K, V, dtype, kw, flush=True)
        o = oracle.verify_chain_warped(inp["target"], inp["draft"], inp["cand"], 0.1, fsd.DIV_TV, fsd.SAMPLE, 9, 4, **kw)
        for rep in range(2):
            out = fsd.fsd_verify_chain_warped(dev["target"], dev["draft"], dev["cand"], 0.1, fsd.DIV_TV, fsd.SAMPLE, 9, 4,
                                              workspace=ws, **kw)
            used, want = fsd.debug_last_selection(), W[0 if "top_k" in kw else 1]
            assert used == want or (kw.get("top_k") == 512 and used < want), (used, want, kw)   # (its lists may want fewer)
            torch_cuda.cuda.synchronize()
            g = pu.host(out, pu.CHAIN_KEYS)
            g["threshold"] = fsd.debug_warp_thresholds(out, B, K, V, code).cpu().numpy()
            check_warped(g, o, 0.1, pu.rel_tol(dtype), f"split selection B={B} V={V} {dtype} {kw}", envelope=pu.Envelope(dtype))


@pytest.mark.parametrize("V,dtype", [(40000, "bf16"), (40003, "bf16"), (40000, "f32"), (40003, "f32")])
def test_split_selection_over_a_tree(torch_cuda, oracle, V, dtype):
    """Every workgroup that shares a row finds the row for itself, over a tree by its deepest accepted path."""
    B, N = 4, 14
    inp = _random_tree_inputs(np.random.default_rng(V), B, N, V, dtype)
    d = pu.to_dev(inp, ("target", "draft", "node_tokens", "parent"))
    code = fsd.BF16 if dtype == "bf16" else fsd.F32
    for kw in (dict(temperature=0.7, top_k=50, top_p=0.9), dict(top_p=0.8)):
        what = f"split selection over a tree V={V} {dtype} {kw}"
        print(what, flush=True)
        out = fsd.fsd_verify_tree_warped(d["target"], d["draft"], d["node_tokens"], d["parent"], N, 0.12, fsd.DIV_JS, fsd.SAMPLE, 5, 2, **kw)
        assert fsd.debug_last_selection() > 1, what
        torch_cuda.cuda.synchronize()
        g = pu.host(out, pu.TREE_KEYS)
        thr = fsd.debug_warp_thresholds(out, B, N, V, code).cpu().numpy()
        o = oracle.verify_tree_warped(inp["target"], inp["draft"], inp["node_tokens"], inp["parent"], N, 0.12, fsd.DIV_JS, fsd.SAMPLE, 5, 2, **kw)
        assert (g["row_status"] == 0).all() and (o["row_status"] == 0).all(), what
        near = pu.near_threshold(o["divs"], 0.12)
        for b in range(B):
            if not (g["path_nodes"][b] == o["path_nodes"][b]).all():
                assert near[b].any(), what
                continue
            if o["slack"][b] >= 1e-5:
                assert thr[b] == o["threshold"][b], f"{what}: cut[{b}] gpu {thr[b]} oracle {o['threshold'][b]}"
            if not (g["out_tokens"][b] == o["out_tokens"][b]).all():
                assert o["slack"][b] < 1e-5 or o["gap"][b] < 1e-6, f"{what}: tokens[{b}]"


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("V", [40000, 40003, 300])
def test_selection_on_an_unusable_row(torch_cuda, dtype, V):
    """The row after the last candidate, which the reduction does not read: NaN, +inf or no entry above -inf is found
    by the draw and reported for that sequence alone, whichever way its cut was looked for."""
    B, K = 6, 13
    inp = synth.chain_inputs(B, K, V, dtype, "peaked", 1.0, seed=31)
    put = (lambda x: synth.to_bf16_bits(np.full(1, x, np.float32))[0]) if dtype == "bf16" else np.float32
    inp["target"][1, K, V // 2] = put(np.nan)
    inp["target"][2, K, V - 1] = put(np.inf)
    inp["target"][3, K] = put(-np.inf)
    inp["target"][4, K, 1:] = put(-np.inf)                             # one entry: the token
    d = pu.to_dev(inp, ("target", "draft", "cand"))
    for kw in (dict(top_k=40, top_p=0.9), dict(top_k=40), dict(top_p=0.9), dict(top_k=V - 2)):
        print("unusable row", V, dtype, kw, flush=True)
        out = fsd.fsd_verify_chain_warped(d["target"], d["draft"], d["cand"], float("inf"), fsd.DIV_TV, fsd.SAMPLE, 9, 4, **kw)
        assert V < 40000 or kw.get("top_k", 0) > 512 or fsd.debug_last_selection() > 1
        torch_cuda.cuda.synchronize()
        g = pu.host(out, pu.CHAIN_KEYS)
        assert list(g["row_status"]) == [0] + 3 * [fsd.ROW_NONFINITE] + [0, 0], kw
        assert (g["accept_len"] == np.array([K, 0, 0, 0, K, K])).all() and (g["out_tokens"][1:4] == -1).all()
        assert g["out_tokens"][4, K] == 0 and (g["out_tokens"][[0, 5], K] >= 0).all()


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_selection_wait_expires_cleanly(torch_cuda, oracle, dtype):
    """The workgroups that share a row under top-p wait for each other's range with a poll budget.  With one of zero
    the kernel ends and the call flags every sequence, unless all words were there at the first look; the
    next call on the same workspace is right."""
    B, K, V = 4, 13, 40003
    inp = synth.chain_inputs(B, K, V, dtype, "peaked", 1.0, seed=21)
    dev = pu.to_dev(inp, ("target", "draft", "cand"))
    code = fsd.BF16 if dtype == "bf16" else fsd.F32
    ws = torch_cuda.empty(fsd.fsd_workspace_bytes(B, K, V, code) + 256, dtype=torch_cuda.uint8, device="cuda")
    o = oracle.verify_chain_warped(inp["target"], inp["draft"], inp["cand"], 0.1, fsd.DIV_TV, fsd.SAMPLE, 9, 4, top_p=0.9)

    def call():
        out = fsd.fsd_verify_chain_warped(dev["target"], dev["draft"], dev["cand"], 0.1, fsd.DIV_TV, fsd.SAMPLE, 9, 4,
                                          workspace=ws, top_p=0.9)
        assert fsd.debug_last_selection() > 1
        torch_cuda.cuda.synchronize()
        g = pu.host(out, pu.CHAIN_KEYS)
        g["threshold"] = fsd.debug_warp_thresholds(out, B, K, V, code).cpu().numpy()
        return g

    for rep in range(3):
        prev = fsd.debug_set_selection_spin_limit(0)
        try:
            g = call()
        finally:
            fsd.debug_set_selection_spin_limit(prev)
        flagged = (g["row_status"] & fsd.ROW_INTERNAL) != 0
        print("selection wait", dtype, "flagged", flagged, flush=True)
        assert flagged.all() or not flagged.any()
        if flagged.all():
            assert (g["accept_len"] == 0).all() and (g["out_tokens"] == -1).all()
        else:
            check_warped(g, o, 0.1, pu.rel_tol(dtype), f"zero poll budget, nothing expired {dtype}", envelope=pu.Envelope(dtype))
        g = call()
        check_warped(g, o, 0.1, pu.rel_tol(dtype), f"after restoring the poll budget {dtype}", envelope=pu.Envelope(dtype))


# (the reduction by teams, and in one step of the device)
@pytest.mark.parametrize("small", [False, True])
@pytest.mark.parametrize("tree", [False, True])
def test_failed_reduction_before_the_draw_with_the_selection(torch_cuda, oracle, tree, small):
    """A reduction whose waits have a poll budget of zero, in front of the selection that draws the token: all sequences are flagged, with
    empty outputs, or all are right; the next call on the same workspace is right."""
    B, N, V = 6, 14, 40000
    inp = _random_tree_inputs(np.random.default_rng(8), B, N, V, "bf16")
    dev = pu.to_dev(inp, ("target", "draft", "node_tokens", "parent"))
    ws = torch_cuda.empty(fsd.fsd_workspace_bytes(B, N, V, fsd.BF16) + 256, dtype=torch_cuda.uint8, device="cuda")
    length, keys = ("path_len", pu.TREE_KEYS) if tree else ("accept_len", pu.CHAIN_KEYS)
    args, kw = (0.12, fsd.DIV_JS, fsd.SAMPLE, 5, 2), dict(top_k=50, top_p=0.9, temperature=0.7)
    if tree:
        o = oracle.verify_tree_warped(inp["target"], inp["draft"], inp["node_tokens"], inp["parent"], N, *args, **kw)
    else:
        o = oracle.verify_chain_warped(inp["target"], inp["draft"], inp["node_tokens"], *args, **kw)
    assert not pu.near_threshold(o["divs"], 0.12).any() and (o["slack"] >= 1e-5).all() and (o["gap"] >= 1e-6).all()

    def call():
        if tree:
            out = fsd.fsd_verify_tree_warped(dev["target"], dev["draft"], dev["node_tokens"], dev["parent"], N, *args, workspace=ws, **kw)
        else:
            out = fsd.fsd_verify_chain_warped(dev["target"], dev["draft"], dev["node_tokens"], *args, workspace=ws, **kw)
        assert fsd.debug_last_selection() > 1 and fsd.debug_last_route() == int(small)
        torch_cuda.cuda.synchronize()
        return pu.host(out, keys)

    outputs = [k for k in keys if k in ("accept_len", "path_len", "path_nodes", "out_tokens")]
    prev_small = fsd.debug_set_small_calls(small)
    try:
        for rep in range(3):
            prev = fsd.debug_set_spin_limit(0)
            try:
                g = call()
            finally:
                fsd.debug_set_spin_limit(prev)
            flagged = (g["row_status"] & fsd.ROW_INTERNAL) != 0
            print("failed reduction", tree, small, "flagged", flagged, flush=True)
            assert flagged.all() or (g["row_status"] == 0).all()
            if flagged.all():
                assert (g[length] == 0).all() and all((g[k] == -1).all() for k in outputs if k != length)
            else:
                assert all((g[k] == o[k]).all() for k in outputs)
            g = call()
            assert (g["row_status"] == 0).all() and all((g[k] == o[k]).all() for k in outputs)
    finally:
        fsd.debug_set_small_calls(prev_small)


def _longest_list(row, W, k, inv_temp, VE):
    """The longest list a workgroup of a split top-k leaves: its entries at or above the k-th largest of its 1024
    threads' maxima, of which the upper half of the 32-bit key counts."""
    sv = row.astype(np.float32) * np.float32(inv_temp)
    u = sv.view(np.uint32)
    key = np.where(u >> 31, ~u, u | np.uint32(0x80000000)).astype(np.uint32)
    nslots = -(-len(row) // VE)
    key = np.concatenate([key, np.zeros(nslots * VE - len(row), np.uint32)]).reshape(nslots, VE)
    share = -(-nslots // W)
    longest = 0
    for lo in range(0, nslots, share):
        mine = key[lo: lo + share]
        maxima = np.zeros(1024, np.uint32)
        np.maximum.at(maxima, np.arange(len(mine)) % 1024, mine.max(axis=1))
        bound = np.sort(maxima)[::-1][k - 1] & np.uint32(0xFFFF0000)
        longest = max(longest, int((mine >= bound).sum()))
    return longest


# (4096 keys for all lists of a sequence, each behind its length)
@pytest.mark.parametrize("V,dtype,k,W", [(131073, "bf16", 300, 8), (131073, "bf16", 512, 4), (131073, "bf16", 400, 6),
                                         (65540, "f32", 512, 4), (65540, "f32", 460, 5), (163840, "f32", 512, 1)])
@pytest.mark.parametrize("temperature", [1.0, 0.3])
def test_split_selection_lists_hold_a_large_top_k(torch_cuda, oracle, V, dtype, k, W, temperature):
    """Under a large top-k as few workgroups share a row as their lists need to be long enough, a single one where
    that leaves them more than they can keep of it."""
    rng = np.random.default_rng(V + k)
    B, K, VE = 2, 9, 8 if dtype == "bf16" else 4
    t = (rng.standard_normal((B, K + 1, V), dtype=np.float32) * np.float32(3))
    d = (t[:, :K] + rng.standard_normal((B, K, V), dtype=np.float32) * np.float32(0.3))
    cand = rng.integers(0, V, (B, K)).astype(np.int32)
    rows = t[:, 0]
    inp = dict(target=t, draft=d, cand=cand)
    if dtype == "bf16":
        inp = dict(target=synth.to_bf16_bits(t), draft=synth.to_bf16_bits(d), cand=cand)
        rows = (inp["target"][:, 0].astype(np.uint32) << 16).view(np.float32)
    kw = dict(temperature=temperature, top_k=k)
    print("large top-k", V, dtype, kw, flush=True)
    g = run_warped(torch_cuda, inp, -1.0, fsd.DIV_TV, fsd.SAMPLE, 9, 4, **kw)   # (row 0 is drawn from)
    used = fsd.debug_last_selection()
    if used > 1:
        longest = max(_longest_list(r, used, k, np.float32(1.0 / temperature), VE) for r in rows)
        print("workgroups", used, "longest list", longest, "room", 4096 // used - 1, flush=True)
        assert longest <= 4096 // used - 1
    assert used == W
    o = oracle.verify_chain_warped(inp["target"], inp["draft"], inp["cand"], -1.0, fsd.DIV_TV, fsd.SAMPLE, 9, 4, **kw)
    check_warped(g, o, -1.0, pu.rel_tol(dtype), f"large top-k V={V} {dtype} {kw}", envelope=pu.Envelope(dtype))


# 128 sequences: 8 workgroups a row; a share's last round has slots for one lane, one wavefront, one lane more, ...
@pytest.mark.parametrize("share", [255, 256, 257, 319, 320, 321, 511, 512, 513, 577])
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_shares_of_a_draw(torch_cuda, oracle, share, dtype):
    """The draw where a share's last round is all, part or none of a wavefront's, with the last share a slot shorter."""
    B, V = 128, (8 * share - 1) * (8 if dtype == "bf16" else 4)
    inp = synth.chain_inputs(B, 1, V, dtype, "gauss2", 1.0, seed=share)
    for kw in (dict(mode=fsd.SAMPLE), dict(mode=fsd.GREEDY)):
        g = run_chain(torch_cuda, inp, -1.0, fsd.DIV_TV, kw["mode"], seed=5, offset=2)
        o = oracle.verify_chain(inp["target"], inp["draft"], inp["cand"], -1.0, fsd.DIV_TV, kw["mode"], seed=5, offset=2)
        pu.check_chain(g, o, -1.0, pu.rel_tol(dtype), f"share {share} {dtype} {kw}", envelope=pu.Envelope(dtype))
    g = run_warped(torch_cuda, inp, -1.0, fsd.DIV_TV, fsd.SAMPLE, 5, 2, temperature=0.7)
    o = oracle.verify_chain_warped(inp["target"], inp["draft"], inp["cand"], -1.0, fsd.DIV_TV, fsd.SAMPLE, 5, 2, temperature=0.7)
    check_warped(g, o, -1.0, pu.rel_tol(dtype), f"share {share} {dtype} warped", cut_active=False, envelope=pu.Envelope(dtype))


# 5 wavefronts a compute unit (1280 on 256 of them) with 1024 entries of a binary32 row each
@both_routes
@pytest.mark.parametrize("B,K,V", [(1, 4, 32000), (10, 4, 32000), (11, 4, 32000), (1, 8, 128256), (1, 1, 262144), (1, 1, 262145), (40, 8, 4096)])
@pytest.mark.parametrize("div", [fsd.DIV_JS, fsd.DIV_TV, fsd.DIV_KL])
def test_small_binary32_calls(torch_cuda, oracle, B, K, V, div):
    """Both sides of the line where a binary32 call takes half the slots per lane, and the largest team (256)."""
    inp = synth.chain_inputs(B, K, V, "f32", "gauss2", 0.5, seed=V % 97)
    g = run_chain(torch_cuda, inp, 0.1, div, seed=5, offset=2)
    o = oracle.verify_chain(inp["target"], inp["draft"], inp["cand"], 0.1, div, seed=5, offset=2)
    pu.check_chain(g, o, 0.1, 1e-5, f"small binary32 B={B} K={K} V={V} div={div}", envelope=pu.Envelope("f32"))
    if div == fsd.DIV_JS:
        d = pu.to_dev(inp, ("target", "draft", "cand"))
        out = fsd.sd_verify_chain(d["target"], d["draft"], d["cand"], seed=5, offset=2)
        torch_cuda.cuda.synchronize()
        o = oracle.sd_verify_chain(inp["target"], inp["draft"], inp["cand"], seed=5, offset=2)
        check_sd(pu.host(out, pu.SD_KEYS), o, f"small binary32 SD B={B} K={K} V={V}")


def test_routes_under_capture(torch_cuda):
    """Calls with a split selection, over a tree with the walk, on ragged rows and on a small binary32 batch, recorded
    into a graph: three replays, with the program's own eager calls in between, each equal to the eager result."""
    torch = torch_cuda
    c = pu.to_dev(synth.chain_inputs(4, 13, 40004, "bf16", "peaked", (0.25, 2.0), seed=12), ("target", "draft", "cand"))
    r = pu.to_dev(synth.chain_inputs(3, 4, 40005, "bf16", "peaked", 1.0, seed=13), ("target", "draft", "cand"))
    f = pu.to_dev(synth.chain_inputs(2, 4, 32000, "f32", "gauss2", 0.5, seed=14), ("target", "draft", "cand"))
    t = pu.to_dev(_random_tree_inputs(np.random.default_rng(5), 3, 9, 9000, "bf16"), ("target", "draft", "node_tokens", "parent"))
    calls = [
        lambda **k: fsd.fsd_verify_chain_warped(c["target"], c["draft"], c["cand"], 0.1, seed=4, offset=9, temperature=0.7,
                                                top_k=50, top_p=0.9, **k),
        lambda **k: fsd.fsd_verify_chain_warped(c["target"], c["draft"], c["cand"], 0.1, seed=4, offset=9, top_p=0.9, **k),
        lambda **k: fsd.fsd_verify_chain(r["target"], r["draft"], r["cand"], 0.1, seed=4, offset=9, **k),
        lambda **k: fsd.fsd_verify_chain(f["target"], f["draft"], f["cand"], 0.1, seed=4, offset=9, **k),
        lambda **k: fsd.sd_verify_tree(t["target"], t["draft"], t["node_tokens"], t["parent"], 9, seed=4, offset=9, **k),
    ]
    eager = []
    for i, call in enumerate(calls):
        eager.append(call())
        assert i > 1 or fsd.debug_last_selection() > 1
    torch.cuda.synchronize()
    want = [pu.host(e, [k for k in e if k != "_workspace"]) for e in eager]
    keep = [dict(out={k: torch.empty_like(v) for k, v in e.items() if k != "_workspace"},
                 workspace=torch.empty_like(e["_workspace"]).random_(0, 256)) for e in eager]
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        for call, k in zip(calls, keep):
            call(**k)
    torch.cuda.current_stream().wait_stream(side)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        for call, k in zip(calls, keep):
            call(**k)
    for rep in range(3):
        for k in keep:
            for name, v in k["out"].items():
                if name != "_workspace":
                    v.fill_(-7)
        for call in calls:
            call()
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        for w, k in zip(want, keep):
            for name, v in w.items():
                assert np.array_equal(k["out"][name].cpu().numpy(), v, equal_nan=True), (rep, name)


def test_replays_on_other_inputs(torch_cuda):
    """A replay has the number of the call that was recorded, and so had the replay before it: its words must not count
    again.  Other logits and tokens between the replays, on the recorded call's own workspace, and an eager call on that
    workspace before the last two: every replay equals, bit for bit, an eager call on the same inputs elsewhere.  One launch, the one-step
    reduction with its words in the arrival slots and in the place of the exchange words, calls in one launch whose replays take the
    reduction, the persistent teams, and the calls with kernels between reduction and draw."""
    torch = torch_cuda
    warp = dict(temperature=0.8, top_k=40, top_p=0.9)
    calls = [  # call, B, rows, V, dtype, divergence, more arguments, route, and the recorded call's where it is another
        ("chain", 3, 8, 128256, torch.bfloat16, fsd.DIV_JS, {}, (2, 1)), ("chain", 12, 5, 32000, torch.float32, fsd.DIV_JS, {}, (2, 1)),
        ("tree", 1, 30, 32001, torch.float32, fsd.DIV_KL, {}, (2, 1)), ("tree", 1, 16, 32000, torch.bfloat16, fsd.DIV_KL, {}, 2),
        ("chain", 4, 8, 64000, torch.float32, fsd.DIV_TV, {}, 2),
        ("chain", 2, 4, 32000, torch.float32, fsd.DIV_JS, {}, 2), ("chain", 3, 7, 32001, torch.bfloat16, fsd.DIV_TV, {}, 2),
        ("chain", 3, 5, 20000, torch.bfloat16, fsd.DIV_KL, {}, 2), ("tree", 2, 9, 9000, torch.bfloat16, fsd.DIV_JS, {}, 2),
        ("rfsd", 2, 5, 32000, torch.bfloat16, fsd.DIV_JS, {}, 1), ("chain", 16, 5, 64000, torch.bfloat16, fsd.DIV_JS, {}, 1),
        ("chain", 600, 5, 1500, torch.float32, fsd.DIV_KL, {}, 1), ("warped", 3, 4, 40004, torch.bfloat16, fsd.DIV_JS, warp, 1),
        ("warped", 4, 13, 40004, torch.bfloat16, fsd.DIV_JS, dict(top_p=0.9), 1),
        ("chain", 16, 5, 128259, torch.bfloat16, fsd.DIV_JS, {}, 0), ("sd", 3, 5, 32000, torch.float32, None, {}, 0),
        ("sd_tree", 2, 9, 9000, torch.bfloat16, None, {}, 0)]
    gen = torch.Generator(device="cuda")
    gen.manual_seed(3)

    def inputs(call, B, rows, V, dtype):
        d = dict(target=torch.randn((B, rows + 1, V), generator=gen, device="cuda").mul_(3).to(dtype))
        # (the next row's noise differs from set to set: other divergences, lengths and tokens)
        spread = 0.2 + 1.5 * torch.rand((B, rows, 1), generator=gen, device="cuda")
        d["draft"] = (d["target"][:, :rows].float() + spread * torch.randn((B, rows, V), generator=gen, device="cuda")).to(dtype)
        d["tokens"] = torch.randint(0, V, (B, rows), generator=gen, device="cuda", dtype=torch.int32)
        if "tree" in call:
            d["parent"] = torch.tensor([[-1] + [int(torch.randint(-1, j, (1,))) for j in range(1, rows)] for _ in range(B)],
                                       dtype=torch.int32, device="cuda")
        return d

    def run(call, d, div, more, **keep):
        rnd = dict(seed=4, offset=9, **keep)
        rows, T = d["draft"].shape[1], {fsd.DIV_JS: 0.05, fsd.DIV_TV: 0.2, fsd.DIV_KL: 0.2}.get(div)
        if call == "chain":
            return fsd.fsd_verify_chain(d["target"], d["draft"], d["tokens"], T, div, **rnd)
        if call == "warped":
            return fsd.fsd_verify_chain_warped(d["target"], d["draft"], d["tokens"], T, div, **more, **rnd)
        if call == "rfsd":
            return fsd.rfsd_verify_chain(d["target"], d["draft"], d["tokens"], T, div, **rnd)
        if call == "tree":
            return fsd.fsd_verify_tree(d["target"], d["draft"], d["tokens"], d["parent"], rows, T, div, **rnd)
        if call == "sd":
            return fsd.sd_verify_chain(d["target"], d["draft"], d["tokens"], **rnd)
        return fsd.sd_verify_tree(d["target"], d["draft"], d["tokens"], d["parent"], rows, **rnd)

    for call, B, rows, V, dtype, div, more, route in calls:
        print("replays", call, B, rows, V, dtype, div, more, flush=True)
        sets = [inputs(call, B, rows, V, dtype) for _ in range(3)]
        own = {k: v.clone() for k, v in sets[0].items()}
        first = run(call, own, div, more)
        eager, recorded = route if isinstance(route, tuple) else (route, route)
        assert fsd.debug_last_route() == eager
        out = {k: torch.empty_like(v) for k, v in first.items() if k != "_workspace"}
        names = list(out)
        ws = torch.empty_like(first["_workspace"]).random_(0, 256)
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            run(call, own, div, more, out=out, workspace=ws)
        assert fsd.debug_last_route() == recorded
        seen = []
        for rep in range(6):
            for k, v in sets[rep % 3].items():
                own[k].copy_(v)
            for k in names:
                out[k].fill_(-7)
            want = run(call, sets[rep % 3], div, more)
            if rep >= 4:
                run(call, sets[(rep + 1) % 3], div, more, workspace=ws)
            torch.cuda.synchronize()
            graph.replay()
            torch.cuda.synchronize()
            for k in names:
                assert np.array_equal(out[k].cpu().numpy(), want[k].cpu().numpy(), equal_nan=True), (call, rep, k)
            seen.append(out["out_tokens"].cpu().numpy())
        assert not np.array_equal(seen[0], seen[1]) and np.array_equal(seen[0], seen[3])


# up to 64 positions or nodes are decided by a wavefront, more by the workgroup; V: one, two and several shares of a draw
@both_routes
@pytest.mark.parametrize("rows,V,dtype", [(1, 700, "bf16"), (2, 1025, "f32"), (63, 2056, "bf16"), (64, 4100, "bf16"), (64, 1028, "f32"),
                                          (65, 4096, "bf16"), (65, 1029, "f32"), (130, 520, "f32")])
def test_acceptance_around_a_wavefront_of_rows(torch_cuda, oracle, rows, V, dtype):
    """Prefixes and paths that end at the first, an inner and the last position, or node 63, 64 and 65 of a tree; malformed
    and too deep trees; a sequence with an unusable row beside good ones."""
    rng = np.random.default_rng(rows * 1000 + V)
    B, tol = 4, pu.rel_tol(dtype)
    inp = _random_tree_inputs(rng, B, rows, V, dtype, noise=(0.2, 0.6))
    inp["parent"][1] = np.arange(-1, rows - 1)                       # a chain: the deepest tree there is
    chain = dict(target=inp["target"], draft=inp["draft"].copy(), cand=inp["node_tokens"])
    chain["draft"][:] = chain["target"][:, :rows]                    # equal rows (accepted at any T >= 0) ...
    for b, first in enumerate((0, rows // 2, rows - 1)):             # ... up to one that is not
        chain["draft"][b, first] = chain["target"][b, first][::-1]
    for mode in (fsd.SAMPLE, fsd.GREEDY):
        print("acceptance", rows, V, dtype, mode, flush=True)
        g = run_chain(torch_cuda, chain, 0.01, fsd.DIV_TV, mode, seed=5, offset=2)
        o = oracle.verify_chain(chain["target"], chain["draft"], chain["cand"], 0.01, fsd.DIV_TV, mode, seed=5, offset=2)
        assert list(o["accept_len"]) == [0, rows // 2, rows - 1, rows]
        pu.check_chain(g, o, 0.01, tol, f"acceptance chain rows={rows} {dtype}", envelope=pu.Envelope(dtype))
        for T in (-1.0, float(np.median(o["divs"])), 1e9):
            g = run_tree(torch_cuda, inp, T, fsd.DIV_TV, rows, mode, seed=5, offset=2)
            ot = oracle.verify_tree(inp["target"], inp["draft"], inp["node_tokens"], inp["parent"], rows, T, fsd.DIV_TV, mode, seed=5, offset=2)
            pu.check_tree(g, ot, T, tol, f"acceptance tree rows={rows} {dtype} T={T}", envelope=pu.Envelope(dtype))
    d = pu.to_dev(chain, ("target", "draft", "cand"))
    out = fsd.sd_verify_chain(d["target"], d["draft"], d["cand"], seed=5, offset=2)
    torch_cuda.cuda.synchronize()
    o = oracle.sd_verify_chain(chain["target"], chain["draft"], chain["cand"], seed=5, offset=2)
    check_sd(pu.host(out, pu.SD_KEYS), o, f"acceptance SD rows={rows} {dtype}")
    if rows > 2:
        bad = dict(inp, parent=inp["parent"].copy())
        bad["parent"][0, rows - 1] = rows - 1                        # its own parent
        g = run_tree(torch_cuda, bad, 1e9, fsd.DIV_TV, rows - 1, seed=5, offset=2)
        o = oracle.verify_tree(bad["target"], bad["draft"], bad["node_tokens"], bad["parent"], rows - 1, 1e9, fsd.DIV_TV, seed=5, offset=2)
        assert o["row_status"][0] == fsd.ROW_BAD_PARENT and o["row_status"][1] == fsd.ROW_TOO_DEEP
        assert list(g["row_status"]) == list(o["row_status"])
        assert (g["path_len"][:2] == 0).all() and (g["path_nodes"][:2] == -1).all() and (g["out_tokens"][:2] == -1).all()
        pu.check_tree({k: v[2:] for k, v in g.items()}, {k: v[2:] for k, v in o.items()}, 1e9, tol,
                      f"acceptance beside malformed rows={rows} {dtype}", envelope=pu.Envelope(dtype))
        spoilt = dict(inp, draft=inp["draft"].copy())
        spoilt["draft"][2, rows - 1, 1] = np.uint16(0x7FC0) if dtype == "bf16" else np.float32(np.nan)
        g = run_tree(torch_cuda, spoilt, 1e9, fsd.DIV_TV, rows, seed=5, offset=2)
        assert list(g["row_status"]) == [0, 0, fsd.ROW_NONFINITE, 0] and g["path_len"][2] == 0


# A call in one launch: 2, 4 and 8 slots a lane and the team's limit of 64, the wavefronts up to which it takes 2, one entry behind a
# slot; the rows, entries and bytes up to which a call takes a form, and one beyond.  Routes under JS, TV and KL, then those of
# reducible FSD, then that of a tree under JS where it is another: 2 one launch, 1 the one-step reduction with the sampler
# behind it, 0 the persistent teams
@pytest.mark.parametrize("B,K,V,dtype,routes", [
    (1, 2, 65536, "bf16", "222110"), (1, 2, 65537, "bf16", "222110"), (1, 2, 131073, "bf16", "222110"), (1, 1, 262144, "bf16", "222110"),
    (1, 1, 262145, "bf16", "000000"), (1, 2, 32768, "f32", "222111"), (1, 2, 32769, "f32", "222111"), (1, 2, 65537, "f32", "222111"),
    (1, 1, 131072, "f32", "222111"), (1, 1, 131073, "f32", "000000"), (4, 5, 32000, "bf16", "222110"), (3, 7, 32001, "bf16", "222110"),
    (2, 5, 32001, "f32", "222111"), (3, 4, 32000, "f32", "222111"), (2, 16, 40001, "bf16", "220110"), (1, 32, 520, "bf16", "222110"),
    (1, 33, 520, "bf16", "110110"), (1, 64, 520, "bf16", "110110"), (1, 65, 520, "bf16", "110110"), (1, 32, 520, "f32", "222111"), (1, 65, 520, "f32", "101111"), (64, 1, 1025, "f32", "222111"),
    (13, 5, 1025, "f32", "222111"), (3, 1, 8, "bf16", "222110"), (3, 1, 5, "f32", "222111"), (2, 130, 603, "f32", "101111"),
    (3, 17, 20000, "bf16", "222110"), (3, 19, 20000, "bf16", "220110"), (1, 30, 63550, "bf16", "220110"), (1, 30, 70000, "bf16", "100110"),
    (1, 33, 63544, "bf16", "110110"), (1, 33, 63552, "bf16", "100110"), (1, 33, 63553, "bf16", "110110"), (7, 2, 262144, "bf16", "110110"), (1, 33, 31775, "f32", "101111"), (1, 33, 31776, "f32", "001111"),
    (1, 32, 63551, "f32", "001111"), (1, 33, 63551, "f32", "111111"), (1, 33, 98304, "f32", "111111"), (1, 33, 98305, "f32", "101111"),
    (1, 48, 98304, "f32", "111111"), (1, 49, 98300, "f32", "101101"), (8, 2, 262144, "bf16", "100110"), (8, 2, 262145, "bf16", "000000"),
    (4, 8, 131072, "bf16", "100110"), (4, 9, 131072, "bf16", "1001100"), (4, 9, 131073, "bf16", "100100"), (2, 20, 131072, "bf16", "1001000"),
    (1, 41, 131072, "bf16", "000100"), (1, 41, 98308, "f32", "111111"), (1, 16, 128256, "f32", "201111"), (1, 17, 128256, "f32", "101111"), (1, 64, 98304, "bf16", "100100"),
    (1, 65, 98304, "bf16", "000000"), (7, 11, 47744, "bf16", "200110")])
def test_small_calls(torch_cuda, oracle, B, K, V, dtype, routes):
    """Chains, and trees of the same sizes, under every divergence, and reducible FSD; masked entries, and a row that
    cannot be used where there is a second sequence."""
    rng = np.random.default_rng(V + 64 * K + B)
    inp = _random_tree_inputs(rng, B, K, V, dtype, noise=(0.3, 0.8))
    if V > 100:
        masked = 0xFF80 if dtype == "bf16" else np.float32(-np.inf)
        inp["target"][:, :, V - 3:] = masked
        inp["draft"][:, :, V - 3:] = masked
        if B > 1:
            inp["target"][B - 1, 0, V // 2] = 0x7FC0 if dtype == "bf16" else np.float32(np.nan)
    chain = dict(target=inp["target"], draft=inp["draft"], cand=inp["node_tokens"])
    tol, env = pu.rel_tol(dtype), pu.Envelope(dtype)
    ways = list(map(int, routes))
    for div, T, way, reducible in zip((fsd.DIV_JS, fsd.DIV_TV, fsd.DIV_KL), (0.06, 0.25, 0.2), ways[:3], ways[3:6]):
        for mode in (fsd.SAMPLE, fsd.GREEDY):
            what = f"one launch B={B} K={K} V={V} {dtype} div={div} mode={mode}"
            g = run_chain(torch_cuda, chain, T, div, mode, seed=3, offset=6)
            assert fsd.debug_last_route() == way, what
            o = oracle.verify_chain(chain["target"], chain["draft"], chain["cand"], T, div, mode, seed=3, offset=6)
            pu.check_chain(g, o, T, tol, what, envelope=env)
            g = run_tree(torch_cuda, inp, T, div, K, mode, seed=3, offset=6)
            assert fsd.debug_last_route() == (ways[6] if div == fsd.DIV_JS and len(ways) > 6 else way), what
            o = oracle.verify_tree(inp["target"], inp["draft"], inp["node_tokens"], inp["parent"], K, T, div, mode, seed=3, offset=6)
            pu.check_tree(g, o, T, tol, what + " tree", envelope=env)
        g = run_rfsd(torch_cuda, chain, T, div, seed=3, offset=6)
        assert fsd.debug_last_route() == reducible
        o = oracle.rfsd_verify_chain(chain["target"], chain["draft"], chain["cand"], T, div, seed=3, offset=6)
        check_rfsd(g, o, T, tol, f"small reducible B={B} K={K} V={V} {dtype} div={div}", envelope=env)


# a wavefront's slice of the small calls is 512 or 1024 entries, of the large ones at most 3072; a row that is not 16-byte aligned
@both_routes
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("V", [20000, 20001])
@pytest.mark.parametrize("base", [-200.0, 0.0])
def test_slices_without_mass(torch_cuda, oracle, dtype, V, base):
    """Whole slices masked, by -inf and by the type's lowest value, in the target's rows, the draft's or both, and in the
    rest of the row logits far below and around zero: a slice without mass is weightless whatever the others' level."""
    B, K = 2, 3
    lowest = np.float32(-3.3895314e38) if dtype == "bf16" else np.finfo(np.float32).min
    for value in (-np.inf, lowest):
        for where in ("target", "draft", "both"):
            inp = synth.chain_inputs(B, K, V, "f32", "gauss2", 0.7, seed=V % 31)
            t, d = inp["target"] + np.float32(base), inp["draft"] + np.float32(base)
            if where != "draft":
                t[:, :, 6000:14000] = value
            if where != "target":
                d[:, :, 6000:14000] = value
            if dtype == "bf16":
                t, d = synth.to_bf16_bits(t), synth.to_bf16_bits(d)
            case = dict(target=t, draft=d, cand=inp["cand"])
            what = f"{dtype} V={V} base={base} {where} masked by {value}"
            print(what, flush=True)
            for div, T in ((fsd.DIV_JS, 0.2), (fsd.DIV_TV, 0.4), (fsd.DIV_KL, 0.8)):
                if div == fsd.DIV_KL and where == "draft" and np.isfinite(value):
                    continue   # (about 1e38, where sums leave binary32's range)
                g = run_chain(torch_cuda, case, T, div, seed=5, offset=2)
                o = oracle.verify_chain(t, d, inp["cand"], T, div, seed=5, offset=2)
                assert (o["row_status"] == 0).all()
                pu.check_chain(g, o, T, pu.rel_tol(dtype), f"{what} div={div}", envelope=pu.Envelope(dtype))
            o = oracle.sd_verify_chain(t, d, inp["cand"], seed=5, offset=2)
            dev = pu.to_dev(case, ("target", "draft", "cand"))
            out = fsd.sd_verify_chain(dev["target"], dev["draft"], dev["cand"], seed=5, offset=2)
            torch_cuda.cuda.synchronize()
            check_sd(pu.host(out, pu.SD_KEYS), o, what)


@both_routes
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("base", [150.0, 0.0, -200.0])
@pytest.mark.parametrize("V,kept", [(40000, 600), (40000, 40), (40003, 20000), (8200, 2)])
def test_sparse_rows(torch_cuda, oracle, dtype, base, V, kept):
    """All but a few entries of every row masked, at places that the two models share, and the rest far above, around and far
    below zero: a lane's, a wavefront's largest logit stands between masked ones, or there is none."""
    B, K = 2, 3
    rng = np.random.default_rng(kept)
    inp = synth.chain_inputs(B, K, V, "f32", "gauss2", 0.7, seed=kept)
    t, d = inp["target"] + np.float32(base), inp["draft"] + np.float32(base)
    for b in range(B):
        at = rng.permutation(V)[kept:]
        t[b, :, at] = -np.inf
        d[b, :, at] = -np.inf
    if dtype == "bf16":
        t, d = synth.to_bf16_bits(t), synth.to_bf16_bits(d)
    case = dict(target=t, draft=d, cand=inp["cand"])
    for div, T in ((fsd.DIV_JS, 0.06), (fsd.DIV_TV, 0.25), (fsd.DIV_KL, 0.25)):
        what = f"{dtype} V={V} kept={kept} base={base} div={div}"
        print(what, flush=True)
        g = run_chain(torch_cuda, case, T, div, seed=5, offset=2)
        o = oracle.verify_chain(t, d, inp["cand"], T, div, seed=5, offset=2)
        assert (o["row_status"] == 0).all()
        pu.check_chain(g, o, T, pu.rel_tol(dtype), what, envelope=pu.Envelope(dtype))


# flat and Zipf-shaped rows from one wavefront's to 64 wavefronts', KL from 0.4 to 3
@pytest.mark.parametrize("kind,sigma,V", [("gauss2", 1.0, 32000), ("gauss2", 1.0, 128256), ("gauss2", 1.0, 250000), ("gauss2", 2.5, 8003),
                                          ("zipf", 2.5, 1000)])
def test_small_kl_is_as_exact_as_in_large_calls(torch_cuda, oracle, kind, sigma, V):
    """Bfloat16 KL against 64 bits in small calls and, the same rows, in the kernel of large ones, whose sums are float64: the rms
    error is no larger.  (Two estimates from 160 pairs or more scatter by 6 % each: 1.2 is two deviations of their ratio.  With
    binary32 sums in the small calls the ratio was 1.3 to 2.2 here.)"""
    K = 4
    B = max(1, min(40, 1100000 // (K * V)))
    err = {True: [], False: []}
    try:
        for seed in range(-(-160 // (B * K))):
            inp = synth.chain_inputs(B, K, V, "bf16", kind, sigma, seed=seed)
            o = oracle.verify_chain(inp["target"], inp["draft"], inp["cand"], 0.1, fsd.DIV_KL)
            for small in err:
                fsd.debug_set_small_calls(small)
                g = run_chain(torch_cuda, inp, 0.1, fsd.DIV_KL)
                assert (fsd.debug_last_route() > 0) == small
                err[small].append((g["divergences"].astype(np.float64) - o["divs"]) / o["divs"])
    finally:
        fsd.debug_set_small_calls(True)
    rms = {small: float(np.sqrt(np.mean(np.concatenate(e) ** 2))) for small, e in err.items()}
    print(kind, sigma, V, "rms error against 64 bits: small calls", rms[True], "large", rms[False], flush=True)
    assert rms[True] <= 1.2 * rms[False]


@pytest.mark.parametrize("V", [5, 3071, 6145, 20000])
@pytest.mark.parametrize("kind", ["log-probabilities", "one slice", "signed zeros", "masked"])
def test_largest_logit_is_negative(torch_cuda, oracle, V, kind):
    """Bfloat16 rows in the kernels of large calls where a wavefront's largest logit is negative, whose packed maximum is taken
    in a second look: all of the row, all but one slice of it, beside signed zeros, between masked entries; a chain, a tree
    whose siblings share target rows, and strict SD."""
    B, K = 2, 5
    rng = np.random.default_rng(V)
    inp = synth.chain_inputs(B, K, V, "f32", "gauss2", 0.7, seed=V)
    t, d = inp["target"], inp["draft"]
    # (masked at the same places: with 3e38 in the draft alone KL is of that size, past binary32's largest number in a sum of logits)
    masked = rng.permutation(V)[: V // 2]
    for x in (t, d):
        x -= x.max(-1, keepdims=True) + np.float32(1.0)
        if kind == "one slice":
            x[..., -min(V, 70):] += np.float32(9.0)
        elif kind == "signed zeros":
            x[..., rng.permutation(V)[: V // 3 + 1]] = -0.0
            x[..., rng.permutation(V)[: V // 3]] = 0.0 if V % 2 else -0.0
        elif kind == "masked":
            x[..., masked] = -np.inf if V % 2 else np.float32(-3.0e38)
    t, d = synth.to_bf16_bits(t), synth.to_bf16_bits(d)
    case = dict(target=t, draft=d, cand=inp["cand"])
    parent = np.broadcast_to(np.array([-1, -1, 0, 0, 2], dtype=np.int32), (B, K)).copy()
    env = pu.Envelope("bf16")
    prev = fsd.debug_set_small_calls(False)
    try:
        for div, T in ((fsd.DIV_JS, 0.06), (fsd.DIV_TV, 0.25), (fsd.DIV_KL, 0.25)):
            what = f"{kind} V={V} div={div}"
            print(what, flush=True)
            g = run_chain(torch_cuda, case, T, div, seed=5, offset=2)
            pu.check_chain(g, oracle.verify_chain(t, d, inp["cand"], T, div, seed=5, offset=2), T, pu.rel_tol("bf16"), what, envelope=env)
            g = run_tree(torch_cuda, dict(target=t, draft=d, node_tokens=inp["cand"], parent=parent), T, div, 4, seed=5, offset=2)
            o = oracle.verify_tree(t, d, inp["cand"], parent, 4, T, div, oracle.SAMPLE, seed=5, offset=2)
            pu.check_tree(g, o, T, pu.rel_tol("bf16"), f"tree {what}", envelope=env)
        dev = pu.to_dev(case, ("target", "draft", "cand"))
        out = fsd.sd_verify_chain(dev["target"], dev["draft"], dev["cand"], seed=5, offset=2)
        torch_cuda.cuda.synchronize()
        check_sd(pu.host(out, pu.SD_KEYS), oracle.sd_verify_chain(t, d, inp["cand"], seed=5, offset=2), f"SD {kind} V={V}")
    finally:
        fsd.debug_set_small_calls(prev)


# two and two steps of teams of 98 and 79 (of 8 slots a lane and of 10), five and four; teams of 75 and 60, of 196 and 157
@pytest.mark.parametrize("B,K,V,eight", [(5, 8, 200000, True), (12, 8, 200000, False), (12, 6, 151936, False), (4, 8, 400004, False)])
def test_binary32_shapes_of_wide_rows(torch_cuda, B, K, V, eight):
    """Which shape a binary32 call of few steps and wide rows takes, and that its results are those of the other one to rounding."""
    torch = torch_cuda
    g = torch.Generator(device="cuda").manual_seed(B)
    t = torch.randn((B, K + 1, V), generator=g, device="cuda") * 2.0
    d = t[:, :K] + torch.randn((B, K, V), generator=g, device="cuda") * 0.5
    cand = torch.zeros((B, K), dtype=torch.int32, device="cuda")
    for div in (fsd.DIV_JS, fsd.DIV_TV, fsd.DIV_KL):
        got, grid = {}, {}
        for slots in (0, 8):
            fsd.debug_set_shape(0, slots)
            try:
                out = fsd.fsd_verify_chain(t, d, cand, 0.1, div, fsd.SAMPLE, 1, 1)
                torch.cuda.synchronize()
            finally:
                fsd.debug_set_shape(0, 0)
            got[slots], grid[slots] = out["divergences"].double(), _last_launch()[0]
        assert (grid[0] == grid[8]) == eight, grid
        assert ((got[0] - got[8]).abs() <= 4e-6 * got[8]).all()


# one member and three, aligned and not; whole members of the single pass's 8 slots
@pytest.mark.parametrize("V", [3071, 6145, 8192])
def test_rows_of_either_sign_one_after_the_other(torch_cuda, oracle, V):
    """A wavefront looks first for the maximum of the sign that its last pair of rows had.  Calls of several rounds, in which rows of logits, of
    log-probabilities, of one in either place, of one slice above zero, of signed zeros, masked and unusable ones follow one another in changing
    order: the first copy against the oracle, the others, which came after other rows, against the first to the bit."""
    torch, B, K, copies = torch_cuda, 8, 13, 100
    rng = np.random.default_rng(V)
    inp = synth.chain_inputs(B, K, V, "f32", "gauss2", 0.7, seed=V)
    t, d = inp["target"], inp["draft"]
    for b in range(B):
        for k in range(K):
            kind = (3 * b + 5 * k) % 8
            if kind in (1, 2, 4, 5):
                t[b, k] -= t[b, k].max() + np.float32(1.0)
            if kind in (1, 3, 4, 5):
                d[b, k] -= d[b, k].max() + np.float32(1.0)
            if kind == 4:
                t[b, k, -70:] += np.float32(9.0)
            if kind == 5:
                t[b, k, rng.permutation(V)[: V // 3]] = 0.0
                d[b, k, rng.permutation(V)[: V // 3]] = -0.0
            if kind == 6:
                masked = rng.permutation(V)[: V // 2]
                t[b, k, masked] = d[b, k, masked] = -np.inf
    d[B - 1, 4, V // 2] = np.nan
    d[B - 1, 9, V // 2] = np.inf
    t, d = synth.to_bf16_bits(t), synth.to_bf16_bits(d)
    parent = np.broadcast_to(np.maximum(np.arange(K) // 3 - 1, -1).astype(np.int32), (B, K)).copy()
    dev = {k: x.repeat(copies, *(1 for _ in x.shape[1:])) for k, x in pu.to_dev(dict(target=t, draft=d, cand=inp["cand"]), ("target", "draft", "cand")).items()}
    parents = torch.from_numpy(parent).cuda().repeat(copies, 1)

    def first(out, keys, tree):
        all_ = out["divergences"].reshape(copies, B, K)[:, : B - 1]
        # (over a tree a row of masked entries may be the first of its siblings or a later one, which takes its sums from the one before: they are
        # rounded in another order then.  Results of the entropy form are exact to 1e-7.)
        if tree:
            assert ((all_ - all_[:1]).abs() <= 1e-6 * (1 + all_.abs())).logical_or(all_ == all_[:1]).all()
        else:
            assert (all_.view(torch.int32) == all_[:1].view(torch.int32)).all()
        assert (out["row_status"].reshape(copies, B) == out["row_status"][:B]).all() and int(out["row_status"][B - 1]) & fsd.ROW_NONFINITE
        return {k: v[: B - 1] for k, v in pu.host(out, keys).items()}

    env, few = pu.Envelope("bf16"), slice(0, B - 1)
    for div, T in ((fsd.DIV_JS, 0.06), (fsd.DIV_TV, 0.25), (fsd.DIV_KL, 0.25)):
        what = f"either sign V={V} div={div}"
        print(what, flush=True)
        out = fsd.fsd_verify_chain(dev["target"], dev["draft"], dev["cand"], T, div, fsd.SAMPLE, 5, 2)
        torch.cuda.synchronize()
        o = oracle.verify_chain(t[few], d[few], inp["cand"][few], T, div, seed=5, offset=2)
        pu.check_chain(first(out, pu.CHAIN_KEYS, False), o, T, pu.rel_tol("bf16"), what, envelope=env)
        out = fsd.fsd_verify_tree(dev["target"], dev["draft"], dev["cand"], parents, 4, T, div, fsd.SAMPLE, 5, 2)
        torch.cuda.synchronize()
        o = oracle.verify_tree(t[few], d[few], inp["cand"][few], parent[few], 4, T, div, oracle.SAMPLE, seed=5, offset=2)
        pu.check_tree(first(out, pu.TREE_KEYS, True), o, T, pu.rel_tol("bf16"), f"tree {what}", envelope=env)
    out = fsd.sd_verify_chain(dev["target"], dev["draft"], dev["cand"], seed=5, offset=2)
    torch.cuda.synchronize()
    got = out["log_ratio"].reshape(copies, B, K)[:, : B - 1].view(torch.int32)
    assert (got == got[:1]).all()
    check_sd({k: v[: B - 1] for k, v in pu.host(out, pu.SD_KEYS).items()}, oracle.sd_verify_chain(t[few], d[few], inp["cand"][few], seed=5, offset=2), f"SD either sign V={V}")


# binary32 rows of whole members of 10 slots a lane (20480, 2560), a slot less, an entry more, a few slots in the last member; 8 slots a
# lane (41000, 41003): two steps of either
@pytest.mark.parametrize("B,K,V", [(16, 15, 20480), (16, 15, 20476), (16, 15, 20481), (100, 15, 2560), (90, 15, 2572), (8, 16, 41000), (8, 16, 41003)])
def test_binary32_teams(torch_cuda, oracle, B, K, V):
    inp = synth.chain_inputs(B, K, V, "f32", "peaked", (0.25, 2.0), seed=V)
    inp["target"][1, 2] = inp["draft"][1, 2]                              # equal rows
    inp["draft"][2, 1, : V // 2] = -np.inf                                # half of a draft row masked
    parent = np.broadcast_to(np.maximum(np.arange(K) // 3 - 1, -1).astype(np.int32), (B, K)).copy()
    env = pu.Envelope("f32")
    prev = fsd.debug_set_small_calls(False)
    try:
        for div, T in ((fsd.DIV_JS, 0.06), (fsd.DIV_TV, 0.25), (fsd.DIV_KL, 0.25)):
            what = f"binary32 teams B={B} K={K} V={V} div={div}"
            print(what, flush=True)
            g = run_chain(torch_cuda, inp, T, div, seed=5, offset=2)
            o = oracle.verify_chain(inp["target"], inp["draft"], inp["cand"], T, div, seed=5, offset=2)
            pu.check_chain(g, o, T, pu.rel_tol("f32"), what, envelope=env)
            g = run_tree(torch_cuda, dict(target=inp["target"], draft=inp["draft"], node_tokens=inp["cand"], parent=parent), T, div, 4, seed=5, offset=2)
            o = oracle.verify_tree(inp["target"], inp["draft"], inp["cand"], parent, 4, T, div, oracle.SAMPLE, seed=5, offset=2)
            pu.check_tree(g, o, T, pu.rel_tol("f32"), f"tree {what}", envelope=env)
    finally:
        fsd.debug_set_small_calls(prev)


# bfloat16 rows of whole members of 8 slots a lane (8192), a slot less and more, rows that are not 16-byte aligned, one member with a slot; 4100
# is below the line in all three calls, so that either side of it is compared
@pytest.mark.parametrize("V,copies", [(8192, 80), (8184, 80), (8200, 80), (8195, 80), (8, 2000), (4100, 20)])
def test_bfloat16_single_pass_teams(torch_cuda, oracle, V, copies):
    """Large calls made of copies of eight sequences: the first copy against the oracle, the others against the first."""
    torch, B, K = torch_cuda, 8, 12
    inp = synth.chain_inputs(B, K, V, "bf16", "peaked", (0.25, 2.0), seed=V)
    inp["target"][1, 2] = inp["draft"][1, 2]                              # equal rows
    inp["target"][3] = synth.to_bf16_bits(np.full((K + 1, V), -2.0, dtype=np.float32))   # negative throughout, all equal
    parent = np.broadcast_to(np.maximum(np.arange(K) // 3 - 1, -1).astype(np.int32), (B, K)).copy()
    dev = pu.to_dev(inp, ("target", "draft", "cand"))
    many = {k: x.repeat(copies, *(1 for _ in x.shape[1:])) for k, x in dev.items()}
    parents = torch.from_numpy(parent).cuda().repeat(copies, 1)
    same = lambda x: x.reshape(copies, B, *x.shape[1:]).view(torch.int32)
    first = lambda out, keys: {k: v[:B] for k, v in pu.host(out, keys).items()}

    out = fsd.sd_verify_chain(many["target"], many["draft"], many["cand"], seed=5, offset=2)
    torch.cuda.synchronize()
    check_sd(first(out, pu.SD_KEYS), oracle.sd_verify_chain(inp["target"], inp["draft"], inp["cand"], seed=5, offset=2), f"SD V={V}")
    assert (same(out["log_ratio"]) == same(out["log_ratio"])[:1]).all()

    env = pu.Envelope("bf16")
    out = fsd.fsd_verify_chain(many["target"], many["draft"], many["cand"], 0.25, fsd.DIV_KL, fsd.SAMPLE, 5, 2)
    torch.cuda.synchronize()
    o = oracle.verify_chain(inp["target"], inp["draft"], inp["cand"], 0.25, fsd.DIV_KL, seed=5, offset=2)
    pu.check_chain(first(out, pu.CHAIN_KEYS), o, 0.25, pu.rel_tol("bf16"), f"KL V={V}", envelope=env)
    assert (same(out["divergences"]) == same(out["divergences"])[:1]).all()

    out = fsd.fsd_verify_tree(many["target"], many["draft"], many["cand"], parents, 4, 0.25, fsd.DIV_KL, fsd.SAMPLE, 5, 2)
    torch.cuda.synchronize()
    o = oracle.verify_tree(inp["target"], inp["draft"], inp["cand"], parent, 4, 0.25, fsd.DIV_KL, oracle.SAMPLE, seed=5, offset=2)
    pu.check_tree(first(out, pu.TREE_KEYS), o, 0.25, pu.rel_tol("bf16"), f"KL tree V={V}", envelope=env)
    assert (same(out["divergences"]) == same(out["divergences"])[:1]).all()

    out = fsd.sd_verify_tree(many["target"], many["draft"], many["cand"], parents, 4, seed=5, offset=2)
    torch.cuda.synchronize()
    o = oracle.sd_verify_tree(inp["target"], inp["draft"], inp["cand"], parent, 4, seed=5, offset=2)
    tree = dict(target=inp["target"], draft=inp["draft"], node_tokens=inp["cand"], parent=parent)
    check_sd_tree(first(out, pu.TREESD_KEYS), o, f"SD tree V={V}", tree)


def _last_launch():
    grid, resident = ctypes.c_int(), ctypes.c_int()
    fsd.library().fsd_debug_last_launch(ctypes.byref(grid), ctypes.byref(resident))
    return grid.value, resident.value


# (trees of 12, or chains of 12; the rounds of its teams that a call of so many rows is)
@pytest.mark.parametrize("tree,B,wide", [(True, 640, False), (True, 2000, False), (True, 3000, True), (False, 640, False), (False, 1500, False), (False, 2100, True)])
def test_bfloat16_kl_takes_the_large_shape_in_large_calls(torch_cuda, oracle, tree, B, wide):
    """KL over bfloat16 rows: the 8-slot shape from 24 rounds of its teams on over trees and 32 over chains, where it is the faster one, and
    the 4-slot shape below; copies of eight sequences, the first copy against the oracle and the others against the first."""
    torch, K, V = torch_cuda, 12, 8192
    inp = synth.chain_inputs(8, K, V, "bf16", "peaked", (0.25, 2.0), seed=3)
    parent = np.broadcast_to(np.maximum(np.arange(K) // 3 - 1, -1).astype(np.int32), (8, K)).copy()
    dev = {k: x.repeat((B + 7) // 8, *(1 for _ in x.shape[1:]))[:B] for k, x in pu.to_dev(inp, ("target", "draft", "cand")).items()}
    parents = torch.from_numpy(parent).cuda().repeat((B + 7) // 8, 1)[:B]
    keys = pu.TREE_KEYS if tree else pu.CHAIN_KEYS

    def call(slots):
        fsd.debug_set_shape(0, slots)
        try:
            if tree:
                out = fsd.fsd_verify_tree(dev["target"], dev["draft"], dev["cand"], parents, 4, 0.25, fsd.DIV_KL, fsd.SAMPLE, 5, 2)
            else:
                out = fsd.fsd_verify_chain(dev["target"], dev["draft"], dev["cand"], 0.25, fsd.DIV_KL, fsd.SAMPLE, 5, 2)
            torch.cuda.synchronize()
        finally:
            fsd.debug_set_shape(0, 0)
        return out, _last_launch()[1]

    out, resident = call(0)
    assert (resident != call(4)[1]) == wide
    first = {k: v[:8] for k, v in pu.host(out, keys).items()}
    if tree:
        o = oracle.verify_tree(inp["target"], inp["draft"], inp["cand"], parent, 4, 0.25, fsd.DIV_KL, oracle.SAMPLE, seed=5, offset=2)
        pu.check_tree(first, o, 0.25, pu.rel_tol("bf16"), f"KL tree B={B}", envelope=pu.Envelope("bf16"))
    else:
        o = oracle.verify_chain(inp["target"], inp["draft"], inp["cand"], 0.25, fsd.DIV_KL, seed=5, offset=2)
        pu.check_chain(first, o, 0.25, pu.rel_tol("bf16"), f"KL B={B}", envelope=pu.Envelope("bf16"))
    got = out["divergences"][: B // 8 * 8].reshape(B // 8, 8, K)
    assert (got == got[:1]).all()


# Rows that begin in the middle of a 32-bit word: every second one of an odd vocabulary (9: two slots, the last of one entry; around whole members of 6 and
# of 4 slots a lane), or all of a tensor that begins there itself (t, d: entries by which the target and the draft are moved); a last slot that is whole
@pytest.mark.parametrize("V,t,d", [(9, 0, 0), (15, 0, 1), (513, 0, 0), (1535, 1, 0), (2047, 0, 0), (2049, 1, 1), (3071, 0, 0), (3073, 0, 1), (6145, 0, 0),
                                   (16, 1, 0), (2048, 0, 1), (3072, 1, 1), (3080, 1, 0), (40007, 0, 0)])
def test_rows_in_the_middle_of_a_word(torch_cuda, oracle, V, t, d):
    torch, B, K = torch_cuda, 9, 7
    inp = synth.chain_inputs(B, K, V, "bf16", "peaked", (0.25, 2.0), seed=V)
    if V > 100:
        inp["target"][1, 2, V - 3:] = 0xFF80
        inp["draft"][1, 2, V - 3:] = 0xFF80
    dev = pu.to_dev(inp, ("target", "draft", "cand"))

    def moved(x, by):
        flat = torch.zeros(x.numel() + by, dtype=x.dtype, device=x.device)
        flat[by:] = x.reshape(-1)
        return flat[by:].view(x.shape)

    target, draft = moved(dev["target"], t), moved(dev["draft"], d)
    tol, env = pu.rel_tol("bf16"), pu.Envelope("bf16")
    prev = fsd.debug_set_small_calls(False)
    try:
        for div, T in ((fsd.DIV_JS, 0.06), (fsd.DIV_TV, 0.25), (fsd.DIV_KL, 0.2)):
            what = f"middle of a word V={V} t={t} d={d} div={div}"
            print(what, flush=True)
            out = fsd.fsd_verify_chain(target, draft, dev["cand"], T, div, fsd.SAMPLE, 5, 2)
            torch.cuda.synchronize()
            o = oracle.verify_chain(inp["target"], inp["draft"], inp["cand"], T, div, seed=5, offset=2)
            pu.check_chain(pu.host(out, pu.CHAIN_KEYS), o, T, tol, what, envelope=env)
            out = fsd.rfsd_verify_chain(target, draft, dev["cand"], T, div, fsd.SAMPLE, 5, 2)
            torch.cuda.synchronize()
            o = oracle.rfsd_verify_chain(inp["target"], inp["draft"], inp["cand"], T, div, seed=5, offset=2)
            check_rfsd(pu.host(out, pu.RFSD_KEYS), o, T, tol, what, envelope=env)
        out = fsd.sd_verify_chain(target, draft, dev["cand"], seed=5, offset=2)
        torch.cuda.synchronize()
        check_sd(pu.host(out, pu.SD_KEYS), oracle.sd_verify_chain(inp["target"], inp["draft"], inp["cand"], seed=5, offset=2), f"SD V={V} t={t} d={d}")
    finally:
        fsd.debug_set_small_calls(prev)


# 1: one entry; 192, 193: the most that is summed up by rank, one more; 500: more candidates than are counted in registers;
# 64, 65 rows: the most a lane each, one more (the draw is then a kernel of its own)
@pytest.mark.parametrize("rows,k", [(13, 1), (13, 2), (13, 192), (13, 193), (13, 500), (64, 40), (65, 40)])
@pytest.mark.parametrize("V,dtype", [(40000, "bf16"), (40003, "f32")])
def test_draw_with_the_selection(torch_cuda, oracle, rows, k, V, dtype):
    """Top-k by several workgroups a row, where the token is drawn by whoever selects: random rows, rows of a few hundred values (ties
    at the cut, and at the nucleus' end), all but 300 entries masked, and the row after the last candidate."""
    B = 4
    rng = np.random.default_rng(rows + k)
    t = (rng.standard_normal((B, rows + 1, V), dtype=np.float32) * np.float32(3))
    t[1] = np.round(t[1] * 16) / 16
    t[2, :, rng.permutation(V)[300:]] = -np.inf
    d = (t[:, :rows] + rng.standard_normal((B, rows, V), dtype=np.float32) * np.float32(0.3))
    d[3] = t[3, :rows]                                                  # everything accepted
    inp = dict(target=t, draft=d, cand=rng.integers(0, V, (B, rows)).astype(np.int32))
    if dtype == "bf16":
        inp.update(target=synth.to_bf16_bits(t), draft=synth.to_bf16_bits(d))
    for kw in (dict(top_k=k), dict(top_k=k, top_p=0.7, temperature=1.3), dict(top_k=k, top_p=0.05), dict(temperature=0.6)):
        what = f"draw with the selection rows={rows} V={V} {dtype} {kw}"
        print(what, flush=True)
        g = run_warped(torch_cuda, inp, 0.005, fsd.DIV_TV, fsd.SAMPLE, 9, 4, **kw)
        assert "top_k" not in kw or fsd.debug_last_selection() > 1
        o = oracle.verify_chain_warped(inp["target"], inp["draft"], inp["cand"], 0.005, fsd.DIV_TV, fsd.SAMPLE, 9, 4, **kw)
        check_warped(g, o, 0.005, pu.rel_tol(dtype), what, cut_active="top_k" in kw, envelope=pu.Envelope(dtype))


@pytest.mark.parametrize("V,kw", [(9000, dict(top_k=300)), (9000, dict(top_k=300, top_p=0.6)), (3000, dict(top_k=700)), (64, dict(top_k=40))])
def test_cut_digits_in_several_quarters(torch_cuda, oracle, V, kw):
    """Logits over [2, 8): their second digit takes all 256 values, and the entries above the bin of the cut lie in the bins of other
    wavefronts.  Many sequences at once, one workgroup each."""
    B = 300
    rng = np.random.default_rng(V)
    t = rng.uniform(2.0, 8.0, (B, 2, V)).astype(np.float32)
    d = (t[:, :1] + rng.standard_normal((B, 1, V), dtype=np.float32) * np.float32(0.3))
    inp = dict(target=t, draft=d, cand=rng.integers(0, V, (B, 1)).astype(np.int32))
    g = run_warped(torch_cuda, inp, 0.01, fsd.DIV_TV, fsd.SAMPLE, 9, 4, **kw)
    assert fsd.debug_last_selection() <= 1
    o = oracle.verify_chain_warped(inp["target"], inp["draft"], inp["cand"], 0.01, fsd.DIV_TV, fsd.SAMPLE, 9, 4, **kw)
    check_warped(g, o, 0.01, pu.rel_tol("f32"), f"cuts V={V} {kw}", envelope=pu.Envelope("f32"))


# two workgroups a sequence: all slots of their threads in use, rows that are not 16-byte aligned, one slot too many
@pytest.mark.parametrize("V,workgroups", [(65536, 2), (65533, 2), (65540, 1)])
@pytest.mark.parametrize("kw", [dict(top_k=40, top_p=0.9, temperature=0.8), dict(top_p=0.8)])
def test_binary32_shares_of_eight_slots(torch_cuda, oracle, V, workgroups, kw):
    """25 copies of four sequences: the first copy against the oracle, the cuts of the others against the first's."""
    inp = synth.chain_inputs(4, 8, V, "f32", "peaked", (0.25, 2.0), seed=V)
    inp["target"][1, :, V // 3:] = -np.inf
    inp["target"][2] = np.round(inp["target"][2] * 4) / 4
    many = {k: np.tile(inp[k], (25,) + (1,) * (inp[k].ndim - 1)) for k in ("target", "draft", "cand")}
    g = run_warped(torch_cuda, many, 0.05, fsd.DIV_JS, fsd.SAMPLE, 9, 4, **kw)
    assert fsd.debug_last_selection() == workgroups
    cuts = g["threshold"].reshape(25, 4)
    assert (cuts == cuts[:1]).all()
    o = oracle.verify_chain_warped(inp["target"], inp["draft"], inp["cand"], 0.05, fsd.DIV_JS, fsd.SAMPLE, 9, 4, **kw)
    check_warped({k: v[:4] for k, v in g.items()}, o, 0.05, pu.rel_tol("f32"), f"shares V={V} {kw}", envelope=pu.Envelope("f32"))


def test_draw_with_the_selection_over_malformed_trees(torch_cuda, oracle):
    """A tree with a parent behind its child, one deeper than the call allows and one as it should be: what the draw with the selection
    reports, and that it leaves nothing of the first two."""
    B, N, V, depth = 3, 14, 40000, 4
    inp = _random_tree_inputs(np.random.default_rng(3), B, N, V, "bf16")
    inp["parent"][:] = np.where(np.arange(N) < 4, -1, np.arange(N) % 4)
    inp["parent"][0, 6] = 9
    inp["parent"][1, 4:9] = np.arange(3, 8)
    d = pu.to_dev(inp, ("target", "draft", "node_tokens", "parent"))
    kw = dict(top_k=50, top_p=0.9)
    out = fsd.fsd_verify_tree_warped(d["target"], d["draft"], d["node_tokens"], d["parent"], depth, 0.12, fsd.DIV_JS, fsd.SAMPLE, 5, 2, **kw)
    assert fsd.debug_last_selection() > 1
    torch_cuda.cuda.synchronize()
    g = pu.host(out, pu.TREE_KEYS)
    o = oracle.verify_tree_warped(inp["target"], inp["draft"], inp["node_tokens"], inp["parent"], depth, 0.12, fsd.DIV_JS, fsd.SAMPLE, 5, 2, **kw)
    assert list(o["row_status"]) == [fsd.ROW_BAD_PARENT, fsd.ROW_TOO_DEEP, 0]
    # (the divergences of a malformed tree's nodes are nobody's: the paths and tokens are what is compared)
    for key in ("row_status", "path_len", "path_nodes", "out_tokens"):
        assert (g[key] == o[key]).all(), key
    assert (g["path_len"][:2] == 0).all() and (g["out_tokens"][:2] == -1).all() and (g["path_nodes"][:2] == -1).all()


# zeros of either sign: so many that every share has more of them than are kept, or 150 of each behind 100 larger entries, where
# the nucleus reaches them only if all are counted; several workgroups a row, and one
@pytest.mark.parametrize("V,dtype,rows,W", [(40000, "bf16", 13, 5), (40003, "f32", 13, 8), (3000, "bf16", 1, 1), (3001, "bf16", 1, 1), (3000, "f32", 1, 1)])
@pytest.mark.parametrize("ones,zeros,kw", [(20, 1500, dict(top_k=60)), (20, 1500, dict(top_k=60, top_p=0.9)), (100, 150, dict(top_k=120, top_p=0.5))])
def test_zeros_of_either_sign_tie(torch_cuda, oracle, V, dtype, rows, W, ones, zeros, kw):
    """A cut at zero keeps +0 and -0 alike, in the draw and in the nucleus' mass."""
    B = 6
    rng = np.random.default_rng(V + ones)
    zeros = min(zeros, V // 3)
    t = rng.uniform(-9, -1, (B, rows + 1, V)).astype(np.float32)
    at = rng.permutation(V)
    t[..., at[:zeros]] = 0.0
    t[..., at[zeros: 2 * zeros]] = -0.0
    t[..., at[2 * zeros: 2 * zeros + ones]] = 1.0
    d = t[:, :rows] + rng.standard_normal((B, rows, V)).astype(np.float32) * np.float32(0.3)
    inp = dict(target=t, draft=d, cand=rng.integers(0, V, (B, rows)).astype(np.int32))
    if dtype == "bf16":
        inp.update(target=synth.to_bf16_bits(t), draft=synth.to_bf16_bits(d))
    for offset in range(3):
        what = f"zeros V={V} {dtype} {kw} offset={offset}"
        print(what, flush=True)
        g = run_warped(torch_cuda, inp, 0.1, fsd.DIV_TV, fsd.SAMPLE, 9, offset, **kw)
        assert fsd.debug_last_selection() == W
        o = oracle.verify_chain_warped(inp["target"], inp["draft"], inp["cand"], 0.1, fsd.DIV_TV, fsd.SAMPLE, 9, offset, **kw)
        assert (o["threshold"] == 0).all() and (o["slack"] > 1e-5).all()
        check_warped(g, o, 0.1, pu.rel_tol(dtype), what, envelope=pu.Envelope(dtype))
        assert (g["out_tokens"] == o["out_tokens"]).all() or (o["gap"] < 1e-6).any(), what


# rows of at most a wavefront's lanes and of more, a tree; one workgroup that draws, and several
@pytest.mark.parametrize("rows,V,tree", [(4, 33000, False), (70, 2000, False), (13, 40003, True)])
def test_temperature_alone_cuts_nothing(torch_cuda, oracle, rows, V, tree):
    """A temperature without top-k and top-p: the cuts left behind are -inf on a workspace that an earlier call has left others on,
    also where nothing is drawn."""
    B = 4
    inp = _random_tree_inputs(np.random.default_rng(V), B, rows, V, "bf16")
    inp["target"][1, :, V // 2] = 0x7FC0                                  # unusable
    dev = pu.to_dev(inp, ("target", "draft", "node_tokens", "parent"))
    ws = torch_cuda.empty(fsd.fsd_workspace_bytes(B, rows, V, fsd.BF16) + 256, dtype=torch_cuda.uint8, device="cuda")
    ws.fill_(0x3F)
    for kw in (dict(top_k=30), dict(temperature=0.7)):
        if tree:
            out = fsd.fsd_verify_tree_warped(dev["target"], dev["draft"], dev["node_tokens"], dev["parent"], rows, 0.1, fsd.DIV_TV, fsd.SAMPLE, 9, 4,
                                             workspace=ws, **kw)
        else:
            out = fsd.fsd_verify_chain_warped(dev["target"], dev["draft"], dev["node_tokens"], 0.1, fsd.DIV_TV, fsd.SAMPLE, 9, 4, workspace=ws, **kw)
        torch_cuda.cuda.synchronize()
        cuts = fsd.debug_warp_thresholds(out, B, rows, V, fsd.BF16).cpu().numpy()
        assert list(out["row_status"].cpu().numpy()) == [0, fsd.ROW_NONFINITE, 0, 0]
        assert (cuts[[0, 2, 3]] > -np.inf).all() == ("top_k" in kw), cuts
    assert (cuts == -np.inf).all() and fsd.debug_last_selection() == 1


@pytest.mark.parametrize("dtype,V", [("bf16", 20000), ("f32", 20000), ("f32", 3001)])
def test_js_of_disjoint_rows_does_not_lean(torch_cuda, dtype, V):
    """Rows of disjoint support, whose divergence is ln 2, in the pointwise form: what rounding makes of it lies on either side.  An entry
    of one row alone weighs its whole probability, whichever row that is; with the next lower number under the logarithm
    (2 - 2^-23 for 2) a row's half of the divergence would lose 6e-8 to 9e-8 of itself, 3e-8 to 4e-8 of the whole.  The mean of 256
    roundings to binary32 (6e-8 apart) is 1e-9 off."""
    B, K = 32, 8
    inp = synth.chain_inputs(B, K, V, "f32", "gauss2", 1.0, seed=V)
    first = np.random.default_rng(V).random(V) < 0.5
    inp["target"][:, :, first] = -np.inf
    inp["draft"][:, :, ~first] = -np.inf
    inp["cand"][:] = np.nonzero(first)[0][0]
    if dtype == "bf16":
        inp.update(target=synth.to_bf16_bits(inp["target"]), draft=synth.to_bf16_bits(inp["draft"]))
    swapped = dict(target=np.concatenate([inp["draft"], inp["draft"][:, :1]], 1), draft=inp["target"][:, :K], cand=np.full_like(inp["cand"], np.nonzero(~first)[0][0]))
    prev = fsd.debug_set_exact_js(True), fsd.debug_set_small_calls(False)
    try:
        for run in (run_chain, run_rfsd):
            err = [(run(torch_cuda, x, 0.1, fsd.DIV_JS, fsd.SAMPLE, 5, 2)["divergences"].astype(np.float64) / np.log(2.0) - 1.0) for x in (inp, swapped)]
            print(run.__name__, dtype, V, [f"{e.mean():+.2e} rms {np.sqrt((e * e).mean()):.2e}" for e in err], flush=True)
            assert all(abs(e.mean()) < 2e-8 for e in err)
    finally:
        fsd.debug_set_exact_js(prev[0])
        fsd.debug_set_small_calls(prev[1])


@pytest.mark.parametrize("V", [64000, 100004])
def test_binary32_large_calls_are_as_exact_as_with_eight_slots(torch_cuda, V):
    """The shape that large binary32 calls take, fewer and larger members of a team, against 64 bits: its error (2-norm over 2-norm, 1024 pairs
    of rows) is no larger than that of the 8-slot shape.  (JS, whose error is mostly the logarithms' own and the same in both, to 1 %.)"""
    torch, B, K = torch_cuda, 64, 16
    g = torch.Generator(device="cuda").manual_seed(7)
    t = torch.randn((B, K + 1, V), generator=g, device="cuda") * 2.0
    d = t[:, :K] + torch.randn((B, K, V), generator=g, device="cuda") * 0.5
    cand = torch.zeros((B, K), dtype=torch.int32, device="cuda")
    exact = {div: [] for div in (fsd.DIV_JS, fsd.DIV_TV, fsd.DIV_KL)}
    for b in range(B):
        lp, lq = torch.log_softmax(t[b, :K].double(), -1), torch.log_softmax(d[b].double(), -1)
        p, q = lp.exp(), lq.exp()
        lm = (0.5 * (p + q)).log()
        exact[fsd.DIV_JS].append(0.5 * (p * (lp - lm) + q * (lq - lm)).sum(-1))
        exact[fsd.DIV_TV].append(0.5 * (p - q).abs().sum(-1))
        exact[fsd.DIV_KL].append((p * (lp - lq)).sum(-1))
    for div, most in ((fsd.DIV_JS, 1.01), (fsd.DIV_TV, 1.0), (fsd.DIV_KL, 1.0)):
        want = torch.stack(exact[div])
        err = {}
        for slots in (0, 8):
            fsd.debug_set_shape(0, slots)
            try:
                out = fsd.fsd_verify_chain(t, d, cand, 0.1, div, fsd.SAMPLE, 1, 1)
                torch.cuda.synchronize()
            finally:
                fsd.debug_set_shape(0, 0)
            err[slots] = float(((out["divergences"].double() - want).norm() / want.norm()).item())
        print(f"binary32 V={V} div={div}: error", err, flush=True)
        assert err[0] <= most * err[8], (div, err)
