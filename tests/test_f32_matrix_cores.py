"""fp32 matrix-core kernel (csrc/f32.hip): its register use on the CPU, and on the GPU every kind at the
edges of its tiles and of the rule that chooses it against the fp64 oracle, at the bar of the other fp32
paths, with NaN in the row padding."""
import numpy as np
import pytest
import torch

import oracle
from _codeobj import kernel_resources, template_args
from paper_2407_09577_amd import workloads

TOL = 1e-5  # row-normwise: fp32 products and chains of at most K / 32 sums


def test_no_spills(tmp_path):
    res = {n: f for n, f in kernel_resources("f32.hip", tmp_path).items() if "f32_mfma_kernel" in n}
    assert res
    assert [n for n, f in res.items() if f.get("private_segment_fixed_size", 0) or f.get("vgpr_spill_count", 0)] == []


def test_vector_tiles_are_built_for_the_kinds_that_can_name_them(tmp_path):
    # f32_kernel is reached by a named configuration alone: linear, GLU, LayerNorm and the two baseline kinds,
    # without run-time g, in its two tile sizes.
    got = sorted(template_args(n) for n in kernel_resources("f32.hip", tmp_path) if "10f32_kernel" in n)
    assert got == sorted([epi, ri, 5 - ri] for epi in range(5) for ri in (1, 4))


def _err(y, ref):
    got = y.cpu().double().numpy()
    assert np.isfinite(got).all()
    return float(np.max(np.abs(got - ref).max(axis=1) / np.abs(ref).max(axis=1)))


# 33 tiles of 16 x 64 and 32 (the few-row kernel), 128 and 127, 384 and 383 tiles of 32 rows; K below one
# block and off every step; ragged rows and columns; one and two rows of wide outputs.
SHAPES = [(16, 4, 33 * 64), (16, 36, 32 * 64), (3, 60, 4099), (1, 132, 65 * 64), (2, 64, 64 * 64), (129, 20, 1000),
          (512, 516, 250), (509, 100, 260), (768, 1028, 1020), (737, 12, 1024), (31, 2048, 777), (250, 4092, 333)]


@pytest.mark.gpu
@pytest.mark.parametrize("M,K,N", SHAPES)
def test_parity_at_edges(M, K, N):
    from paper_2407_09577_amd import flashnorm as fn
    dev = "cuda:0"

    def rows(x):
        big = torch.full((M, K + 12), float("nan"))
        big[:, :K] = x
        return big.to(dev)[:, :K]

    lin = workloads.make("linear", M, K, N, dtype=torch.float32, eps=1e-5, seed=M + K, outlier_frac=0.05)
    ref = oracle.rmsnorm_linear(lin.a, lin.g, lin.W, lin.eps)
    Ws, _, _ = fn.fold_weights(lin.W.to(dev), lin.g.to(dev))
    bias, inv = torch.randn(N, device=dev), torch.empty(M, device=dev)
    y = fn.flashnorm_linear(rows(lin.a), Ws, N, lin.eps, bias=bias, inv_rms=inv)
    assert _err(y, ref + bias.cpu().double().numpy()) <= TOL
    s = 1.0 / torch.sqrt(1e-5 + lin.a.double().square().mean(1))
    assert float((inv.cpu().double() / s - 1).abs().max()) <= 1e-5
    Wp, _, _ = fn.fold_weights(lin.W.to(dev), None)
    y = fn.flashnorm_linear_unfolded(rows(lin.a), lin.g.to(dev), Wp, N, lin.eps)
    assert _err(y, ref) <= TOL

    ln = workloads.make("layernorm", M, K, N, dtype=torch.float32, eps=1e-5, seed=M + K + 1, a_mean=40.0)
    Wl, cs, cb = fn.fold_weights(ln.W.to(dev), ln.g.to(dev), ln.beta.to(dev), colsum=True, c_star=True)
    y = fn.flashnorm_layernorm_linear(rows(ln.a), Wl, cs, cb, N, ln.eps)
    assert _err(y, oracle.layernorm_linear(ln.a, ln.g, ln.beta, ln.W, ln.eps)) <= TOL

    F = N // 2
    glu = workloads.make("glu", M, K, F, dtype=torch.float32, eps=1e-5, seed=M + K + 2)
    Wg, _, _ = fn.fold_weights(glu.W.to(dev), glu.g.to(dev), layout=fn.FN_LAYOUT_GLU)
    y = fn.flashnorm_glu(rows(glu.a), Wg, F, glu.eps)
    assert _err(y, oracle.rmsnorm_swiglu(glu.a, glu.g, glu.W, glu.eps)) <= TOL


@pytest.mark.gpu
@pytest.mark.parametrize("M,Hq,Hkv,h", [(130, 4, 2, 64), (70, 9, 3, 32), (800, 8, 8, 64)])
def test_rotation_and_head_norms(M, Hq, Hkv, h):
    # The kinds whose epilogue exchanges values between lanes, against the forced 64-row tiles (other
    # orders of the fp32 sums: 1e-5 of the row).
    from paper_2407_09577_amd import flashnorm as fn
    dev, K = "cuda:0", 200
    N = (Hq + 2 * Hkv) * h
    w = workloads.make("linear", M, K, N, dtype=torch.float32, seed=M)
    Ws, _, _ = fn.fold_weights(w.W.to(dev), w.g.to(dev))
    cos, sin = (t.to(dev) for t in workloads.rope_tables(512, h))
    pos = workloads.positions(M, 512).to(dev)
    a = w.a.to(dev)
    want = fn.flashnorm_linear(a, Ws, N, w.eps, path=1 << 8)
    y = fn.flashnorm_qkv_rope(a, Ws, Hq, Hkv, h, w.eps, pos, cos, sin, 0.5)
    ref = fn.baseline_rope(want.clone(), Hq, Hkv, h, pos, cos, sin, 0.5)
    assert float(((y - ref).abs().amax(1) / ref.abs().amax(1)).max()) <= 1e-5
    gq, gk = torch.rand(h, device=dev) + 0.5, torch.rand(h, device=dev) + 0.5
    z = fn.flashnorm_qkv_headnorm(a, Ws, Hq, Hkv, h, w.eps, gq, gk, None, 1e-6)
    t = (a.double() * w.g.to(dev).double()) @ w.W.to(dev).double()
    s = (w.eps + a.double().square().mean(1, keepdim=True)).rsqrt()
    heads = t.reshape(M, -1, h)
    nrm = heads / (1e-6 + heads.square().mean(2, keepdim=True)).sqrt()
    nrm[:, :Hq] *= gq.double()
    nrm[:, Hq:Hq + Hkv] *= gk.double()
    nrm[:, Hq + Hkv:] = heads[:, Hq + Hkv:] * s[:, None]
    ref = nrm.flatten(1)
    assert float(((z.double() - ref).abs().amax(1) / ref.abs().amax(1)).max()) <= 1e-5


@pytest.mark.gpu
@pytest.mark.parametrize("M,K,N", [(520, 256, 16), (958, 2380, 6), (1024, 1024, 1), (1009, 516, 11)])
def test_slivers_take_the_few_row_kernel(M, K, N):
    # Outputs of at most 16 columns, 33 to 64 row tiles: the few-row kernel's bits (configuration 3).
    from paper_2407_09577_amd import flashnorm as fn
    w = workloads.make("linear", M, K, N, dtype=torch.float32, eps=1e-5, seed=M)
    Ws, _, _ = fn.fold_weights(w.W.cuda(), w.g.cuda())
    a = w.a.cuda()
    assert torch.equal(fn.flashnorm_linear(a, Ws, N, w.eps), fn.flashnorm_linear(a, Ws, N, w.eps, path=3 << 8))
    # A GLU of at most 16 features, where the rows' pitch is an odd number of 16 bytes.
    g = workloads.make("glu", M, 516, N, dtype=torch.float32, eps=1e-5, seed=N)
    Wg, _, _ = fn.fold_weights(g.W.cuda(), g.g.cuda(), layout=fn.FN_LAYOUT_GLU)
    a = g.a.cuda()
    assert torch.equal(fn.flashnorm_glu(a, Wg, N, g.eps), fn.flashnorm_glu(a, Wg, N, g.eps, path=3 << 8))


@pytest.mark.gpu
def test_more_row_tiles_than_a_grid_dimension():
    # 65536 tiles of 16 rows and a remainder: every kind that has no configuration to name.
    from paper_2407_09577_amd import flashnorm as fn
    M, K = 65536 * 16 + 5, 8
    gen = torch.Generator(device="cuda").manual_seed(3)
    a = torch.randn(M, K, generator=gen, device="cuda")
    g = torch.rand(K, generator=gen, device="cuda") + 0.5
    inv = torch.empty(M, device="cuda")
    x = a.double()
    s = (1e-5 + x.square().mean(1, keepdim=True)).rsqrt()

    def weight(N, use_g):
        W = torch.randn(K, N, generator=gen, device="cuda") * K ** -0.5
        return fn.fold_weights(W, g if use_g else None)[0], (x * g.double()) @ W.double()

    def err(y, ref):
        assert bool(torch.isfinite(y).all())
        return float(((y.double() - ref).abs().amax(1) / ref.abs().amax(1).clamp(min=1e-3)).max())

    Wp, t = weight(20, False)
    assert err(fn.flashnorm_linear_unfolded(a, g, Wp, 20, 1e-5), t * s) <= TOL
    Ws, t = weight(20, True)
    assert err(fn.flashnorm_linear_relu(a, Ws, 20, 1e-5, inv), t.clamp(min=0)) <= TOL
    assert float((inv.double() / s[:, 0] - 1).abs().max()) <= TOL
    pos = torch.arange(M, device="cuda", dtype=torch.int32) % 512
    cos, sin = (v.cuda() for v in workloads.rope_tables(512, 4))
    Ws, t = weight(12, True)
    p = (t * s)[:, :8].reshape(M, 2, 2, 2)
    c, d = cos.double()[pos.long()][:, None], sin.double()[pos.long()][:, None]
    r = torch.stack((p[..., 0] * c - p[..., 1] * d, p[..., 0] * d + p[..., 1] * c), -1).flatten(1)
    r[:, :4] *= 0.5
    y = fn.flashnorm_qkv_rope(a, Ws, 1, 1, 4, 1e-5, pos, cos, sin, 0.5)
    assert err(y, torch.cat((r, (t * s)[:, 8:]), 1)) <= TOL
    Ws, t = weight(24, True)
    one = torch.ones(8, device="cuda")
    h = t.reshape(M, 3, 8)
    n = h / (1e-5 + h.square().mean(2, keepdim=True)).sqrt()
    y = fn.flashnorm_qkv_headnorm(a, Ws, 1, 1, 8, 1e-5, one, one, one, 1e-5)
    assert err(y, n.flatten(1)) <= TOL
