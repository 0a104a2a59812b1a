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


# The kernel of a linear call by the documented rule, from its 16 x 64 and 32 x 64 tiles.
def _kernel(M, K, N):
    nt = (N + 63) // 64
    t16, t32 = nt * ((M + 15) // 16), nt * ((M + 31) // 32)
    if t16 <= 32 or (M <= 2 and nt <= 64) or (N <= 16 and t16 <= 64 and K >= 256):
        return "few rows", t16
    return ("32 rows, 4 waves", t32) if t32 >= 384 else ("16 rows, 4 waves" if t16 >= 128 else "16 rows, 8 waves", t16)


# Both sides of every line of the rule; K below one block and off every step; ragged rows and columns; one and
# two rows of wide outputs.
SHAPES = {(16, 36, 32 * 64): ("few rows", 32), (16, 4, 33 * 64): ("16 rows, 8 waves", 33),
          (16, 20, 127 * 64): ("16 rows, 8 waves", 127), (16, 20, 128 * 64): ("16 rows, 4 waves", 128),
          (32, 12, 383 * 64): ("16 rows, 4 waves", 766), (32, 12, 384 * 64): ("32 rows, 4 waves", 384),
          (2, 64, 64 * 64): ("few rows", 64), (1, 132, 65 * 64): ("16 rows, 8 waves", 65),
          (3, 60, 4099): ("16 rows, 8 waves", 65), (129, 20, 1000): ("16 rows, 4 waves", 144),
          (512, 516, 250): ("16 rows, 4 waves", 128), (509, 100, 260): ("16 rows, 4 waves", 160),
          (768, 1028, 1020): ("32 rows, 4 waves", 384), (737, 12, 1024): ("32 rows, 4 waves", 384),
          (47, 2048, 777): ("16 rows, 8 waves", 39), (250, 4092, 333): ("16 rows, 8 waves", 96),
          (1024, 256, 16): ("few rows", 64), (1025, 256, 16): ("16 rows, 8 waves", 65),
          (1024, 252, 16): ("16 rows, 8 waves", 64), (1024, 256, 17): ("16 rows, 8 waves", 64)}


def test_shapes_hold_both_sides_of_the_rule():
    assert {d: _kernel(*d) for d in SHAPES} == SHAPES


@pytest.mark.gpu
@pytest.mark.parametrize("M,K,N", list(SHAPES))
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


@pytest.mark.gpu
@pytest.mark.parametrize("M,N", [(40, 1024), (1000, 1024)])  # 16-row and 32-row tiles
def test_subnormals(M, N):
    # Subnormal activations, weights, sums and results are kept: small integers times powers of two, whose products
    # and sums are exact in fp32 (the few-row kernel's too).
    from paper_2407_09577_amd import flashnorm as fn
    K = 64
    gen = torch.Generator().manual_seed(N)
    ones = torch.ones(M, device="cuda")
    for ea, ew in ((-149, 100), (100, -149), (-75, -70), (-140, 0)):
        a = torch.ldexp(torch.randint(-7, 8, (M, K), generator=gen).double(), torch.tensor(ea))
        W = torch.ldexp(torch.randint(-7, 8, (K, N), generator=gen).double(), torch.tensor(ew))
        want = (a @ W).float()
        assert torch.equal(want.double(), a @ W) and bool(want.any())
        Wp = fn.fold_weights(W.float().cuda(), None)[0]
        assert torch.equal(fn.rowscale_linear(a.float().cuda(), Wp, N, ones).cpu(), want), (ea, ew)
        few = fn.rowscale_linear(a[:16, :].float().cuda(), fn.fold_weights(W[:, :64].float().cuda(), None)[0], 64, ones[:16])
        assert torch.equal(few.cpu(), want[:16, :64]), (ea, ew)


@pytest.mark.gpu
@pytest.mark.parametrize("M,K,N", [(40, 200, 1000), (130, 1028, 1000), (800, 68, 1020)])
def test_nonfinite_rows_stay_in_their_row(M, K, N):
    # As the oracle: a row with NaN or an infinity is NaN throughout, every other row keeps its bits.
    from paper_2407_09577_amd import flashnorm as fn
    for kind in ("linear", "glu", "layernorm"):
        w = workloads.make(kind, M, K, N // 2 if kind == "glu" else N, dtype=torch.float32, eps=1e-5, seed=M,
                           a_mean=0.5 if kind == "layernorm" else 0.0)
        bad = {0: float("inf"), 18: float("nan"), M - 1: float("-inf")}
        ruined = w.a.clone()
        for r, v in bad.items():
            ruined[r, (5 * r) % K] = v
        ln = kind == "layernorm"
        Ws, cs, cb = fn.fold_weights(w.W.cuda(), w.g.cuda(), w.beta.cuda() if ln else None, colsum=ln, c_star=ln,
                                     layout=fn.FN_LAYOUT_GLU if kind == "glu" else fn.FN_LAYOUT_LINEAR)

        def run(a):
            if ln:
                return fn.flashnorm_layernorm_linear(a.cuda(), Ws, cs, cb, N, w.eps)
            return (fn.flashnorm_glu(a.cuda(), Ws, N // 2, w.eps) if kind == "glu"
                    else fn.flashnorm_linear(a.cuda(), Ws, N, w.eps))

        clean, got = run(w.a), run(ruined)
        good = torch.tensor([r not in bad for r in range(M)], device="cuda")
        assert bool(torch.isnan(got[~good]).all()), kind
        assert bool(torch.isfinite(clean).all()) and torch.equal(got[good], clean[good]), kind
