"""Decode split of narrow outputs (csrc/decode_bf16.hip): one column block per workgroup up to 256 of them,
at its edges, against the fp64 oracle with the bar of the other bf16 paths."""
import numpy as np
import pytest
import torch

import oracle
from paper_2407_09577_amd import workloads

pytestmark = pytest.mark.gpu


def _err(y, ref):
    got = y.float().cpu().double().numpy()
    assert np.isfinite(got).all()
    return float(np.max(np.abs(got - ref).max(axis=1) / np.abs(ref).max(axis=1)))


# One block, the last width of the split and the first past it; K below one block, below one set of the
# eight waves, off every step, and long.
@pytest.mark.parametrize("M,K,N", [(1, 8, 16), (16, 72, 9), (3, 520, 4096), (7, 1032, 4097), (16, 4096, 576),
                                   (2, 8192, 250), (13, 256, 4090)])
def test_parity(M, K, N):
    from paper_2407_09577_amd import flashnorm as fn
    dev = "cuda:0"

    def rows(x):
        big = torch.full((M, K + 8), float("nan"), dtype=torch.bfloat16)
        big[:, :K] = x
        return big.to(dev)[:, :K]

    lin = workloads.make("linear", M, K, N, eps=1e-5, seed=M + K)
    Ws, _, _ = fn.fold_weights(lin.W.to(dev), lin.g.to(dev))
    inv, bias = torch.empty(M, device=dev), torch.randn(N, device=dev)
    y = fn.flashnorm_linear(rows(lin.a), Ws, N, lin.eps, bias=bias, inv_rms=inv)
    assert _err(y, oracle.rmsnorm_linear(lin.a, lin.g, lin.W, lin.eps) + bias.cpu().double().numpy()) <= 2e-2
    s = 1.0 / torch.sqrt(1e-5 + lin.a.double().square().mean(1))
    assert float((inv.cpu().double() / s - 1).abs().max()) <= 1e-5
    ln = workloads.make("layernorm", M, K, N, eps=1e-5, seed=M + K + 1, a_mean=0.5)
    Wl, cs, cb = fn.fold_weights(ln.W.to(dev), ln.g.to(dev), ln.beta.to(dev), colsum=True, c_star=True)
    y = fn.flashnorm_layernorm_linear(rows(ln.a), Wl, cs, cb, N, ln.eps)
    assert _err(y, oracle.layernorm_linear(ln.a, ln.g, ln.beta, ln.W, ln.eps)) <= 2e-2
