"""GPU parity at the sizes and values where a kernel or a rule of its dispatch can go wrong, against the CPU
oracle."""
import numpy as np
import pytest

import paper_2502_20704_amd as fsd
from paper_2502_20704_amd import synth
from tests import parity_util as pu
from tests.test_gpu_parity import check_warped, run_warped

pytestmark = pytest.mark.gpu


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
