"""Middle-row kernel (csrc/mid_kernel.h): its register use and the choice of its workgroup shape on the CPU; on
the GPU the main kinds at the edges of its tiles (row blocks and groups, ragged columns and K, the smallest and
the largest of its range) against the fp64 oracle, and every kind on every workgroup shape against fp64 products
on the GPU, with the row error bar of the other bf16 paths."""
import ctypes
import glob
import os
import re

import numpy as np
import pytest
import torch

import __graft_entry__ as graft
import oracle
from _codeobj import kernel_resources
from paper_2407_09577_amd import workloads

TOL = 2e-2  # row-normwise, bf16: one rounding of W* and one of the output (2 x 2^-8) and the fp32 sums


CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2407_09577_amd", "csrc")
KIND_SOURCES = sorted(os.path.basename(f) for f in glob.glob(os.path.join(CSRC, "mid_kinds_*.hip")))


def test_every_kind_has_its_instances():
    text = "".join(open(os.path.join(CSRC, f)).read() for f in KIND_SOURCES)
    assert sorted(re.findall(r"launch_mid_epi<(EPI_\w+)>", text)) == sorted(
        f"EPI_{k}" for k in ("RMS", "GLU", "LN", "NONE", "GLU_NOSCALE", "REGLU", "BILINEAR", "GLU_DEFER", "RELU_DEFER",
                             "ROWSCALE", "ROPE"))


@pytest.mark.parametrize("source", KIND_SOURCES)
def test_no_spills(source, tmp_path):
    res = kernel_resources(source, tmp_path)
    assert res
    assert [n for n, f in res.items() if f.get("private_segment_fixed_size", 0) or f.get("vgpr_spill_count", 0)
            or f.get("sgpr_spill_count", 0)] == []


def _shape(M, K, N, glu=False):
    """The workgroup shape that the built library takes for a call (-1: the tile kernel)."""
    from paper_2407_09577_amd import flashnorm as fn
    graft.ensure_built()
    choose = getattr(fn.lib(), "_ZN2fn9mid_shapeEiiib")
    choose.argtypes, choose.restype = [ctypes.c_int] * 3 + [ctypes.c_bool], ctypes.c_int
    return choose(M, K, 2 * ((N // 2 + 15) // 16 * 16) if glu else (N + 15) // 16 * 16, glu)


@pytest.mark.parametrize("M,K,N,glu,shape", [
    (17, 4096, 22016, True, 13), (32, 4096, 22016, True, 13), (33, 4096, 22016, False, 14), (48, 4096, 22016, True, 14),
    (49, 4096, 22016, True, 15), (64, 4096, 22016, True, 15), (64, 4096, 22016, False, 15), (65, 4096, 22016, True, 9),
    (32, 8192, 8192, False, 0), (48, 4096, 14336, False, 4), (64, 5120, 15360, False, 7), (32, 4096, 12288, False, 1),
    (17, 7616, 16384, False, 1)])
def test_weight_streams(M, K, N, glu, shape):
    # One row group and 96 MB of weights or more: the smallest shape that holds the rows, six blocks wide with
    # non-temporal loads, unless a narrower one covers the width in one round of workgroups.
    assert _shape(M, K, N, glu) == shape


@pytest.mark.parametrize("M,K,N,glu,shape", [
    (532, 64, 17822, False, -1), (675, 64, 9498, False, -1), (1030, 192, 9090, True, -1), (737, 312, 16450, False, -1), (1527, 16, 20286, True, -1),
    (1306, 256, 3901, False, -1), (1392, 744, 17808, True, -1), (797, 128, 19542, False, 10), (747, 152, 2216, False, 16),
    (23, 64, 16953, False, 2), (333, 4096, 12288, False, 17)])
def test_short_depths(M, K, N, glu, shape):
    # The kernel that is faster where the fixed part of every round and the output's stores make up the call.
    assert _shape(M, K, N, glu) == shape


def _err(y, ref):
    got = y.float().cpu().double().numpy()
    assert np.isfinite(got).all()
    return float(np.max(np.abs(got - ref).max(axis=1) / np.abs(ref).max(axis=1)))


# A call that each workgroup shape takes, plain (M, K, N) and GLU (M, K, 2 F): several row groups with a ragged
# last one, a ragged last column tile, K off the 64-deep packing.  The non-temporal shapes take one group and
# 96 MB of weights; shape 17 takes no GLU, and shape 11 is taken by GLUs alone.
SHAPE_CALLS = [
    (0, (35, 40, 257), (59, 40, 258)), (1, (65, 40, 2744), (66, 40, 2756)), (2, (65, 40, 5572), (65, 40, 5572)),
    (3, (133, 112, 1638), (134, 112, 1682)), (4, (1394, 72, 485), (1393, 72, 482)), (5, (65, 40, 8316), (66, 40, 8198)),
    (6, (1407, 1752, 333), (1397, 1944, 322)), (7, (98, 160, 8191), (97, 200, 8168)),
    (8, (101, 1040, 8225), (99, 1048, 8244)), (9, (130, 656, 11416), (129, 552, 11124)),
    (10, (535, 72, 26516), (522, 72, 26362)), (11, None, (198, 5224, 8250)), (12, (521, 40, 21781), (517, 40, 22188)),
    (13, (30, 2888, 16613), (31, 2480, 19332)), (14, (34, 2152, 22315), (33, 2600, 18440)),
    (15, (55, 2520, 19063), (59, 2768, 17350)), (16, (98, 40, 8195), (97, 40, 8268)), (17, (131, 520, 16863), None)]


def test_every_shape_has_its_calls():
    assert [c[0] for c in SHAPE_CALLS] == list(range(18))
    for shape, plain, glu in SHAPE_CALLS:
        if plain:
            assert _shape(*plain) == shape, plain
            assert _shape(*plain[:2], plain[2] // 4 * 4) == shape, plain  # the width that RoPE takes
        if glu:
            assert _shape(*glu, True) == shape, glu


# (M, K, N): one row over the decode range, one over and under whole row blocks, several row groups,
# K below one set, ragged K, ragged and single column tiles, wide streams, the last row count.
SHAPES = [(17, 8, 256), (31, 72, 264), (33, 512, 1000), (48, 576, 2051), (49, 1032, 300), (64, 64, 4096),
          (65, 200, 513), (97, 2048, 640), (128, 136, 12288), (129, 320, 777), (333, 512, 3000), (750, 264, 272),
          (1536, 1024, 257), (40, 4096, 12288)]


@pytest.mark.gpu
@pytest.mark.parametrize("M,K,N", SHAPES)
def test_parity_at_tile_edges(M, K, N):
    from paper_2407_09577_amd import flashnorm as fn
    dev = "cuda:0"
    pad = 24  # activations with padded rows that hold NaN

    def rows(x):
        big = torch.full((M, K + pad), float("nan"), dtype=torch.bfloat16)
        big[:, :K] = x
        return big.to(dev)[:, :K]

    lin = workloads.make("linear", M, K, N, eps=1e-5, seed=M + K, outlier_frac=0.05)
    Ws, _, _ = fn.fold_weights(lin.W.to(dev), lin.g.to(dev))
    inv = torch.empty(M, dtype=torch.float32, device=dev)
    y = fn.flashnorm_linear(rows(lin.a), Ws, N, lin.eps, inv_rms=inv)
    assert _err(y, oracle.rmsnorm_linear(lin.a, lin.g, lin.W, lin.eps)) <= TOL
    s = 1.0 / torch.sqrt(1e-5 + lin.a.double().square().mean(1))
    assert float((inv.cpu().double() / s - 1).abs().max()) <= 1e-5

    ln = workloads.make("layernorm", M, K, N, eps=1e-5, seed=M + K + 1, a_mean=0.5)
    Wl, cs, cb = fn.fold_weights(ln.W.to(dev), ln.g.to(dev), ln.beta.to(dev), colsum=True, c_star=True)
    y = fn.flashnorm_layernorm_linear(rows(ln.a), Wl, cs, cb, N, ln.eps)
    assert _err(y, oracle.layernorm_linear(ln.a, ln.g, ln.beta, ln.W, ln.eps)) <= TOL

    F = (N + 1) // 2
    glu = workloads.make("glu", M, K, F, eps=1e-5, seed=M + K + 2)
    Wg, _, _ = fn.fold_weights(glu.W.to(dev), glu.g.to(dev), layout=fn.FN_LAYOUT_GLU)
    y = fn.flashnorm_glu(rows(glu.a), Wg, F, glu.eps)
    assert _err(y, oracle.rmsnorm_swiglu(glu.a, glu.g, glu.W, glu.eps)) <= TOL

    # The kinds without a rounding of their own, held to the tiles' results (another order of the
    # fp32 sums and one bf16 rounding of the output on each side, 2^-9 of the value each): 2^-6 of the row.
    scale = torch.rand(M, device=dev) + 0.5
    x = rows(lin.a)
    tile = fn.FN_PATH_PREFILL | (13 << 8)
    plain = fn.flashnorm_linear(x, Ws, N, 0.0, path=tile).float() * x.float().square().mean(1, keepdim=True).sqrt()
    got = fn.rowscale_linear(x, Ws, N, scale).float()
    want = plain * scale[:, None]
    assert float(((got - want).abs().amax(1) / want.abs().amax(1)).max()) <= 2 ** -6


@pytest.mark.gpu
@pytest.mark.parametrize("M,K,Hq,Hkv,h", [(17, 64, 4, 2, 64), (70, 264, 3, 1, 100), (333, 512, 8, 4, 128), (64, 2048, 32, 8, 128)])
def test_rope_matches_projection_then_rotation(M, K, Hq, Hkv, h):
    from paper_2407_09577_amd import flashnorm as fn
    dev = "cuda:0"
    N = (Hq + 2 * Hkv) * h
    w = workloads.make("linear", M, K, N, eps=1e-6, seed=M)
    Ws, _, _ = fn.fold_weights(w.W.to(dev), w.g.to(dev))
    cos, sin = (t.to(dev) for t in workloads.rope_tables(512, h))
    pos = workloads.positions(M, 512).to(dev)
    bias = torch.randn(N, device=dev)
    y = fn.flashnorm_qkv_rope(w.a.to(dev), Ws, Hq, Hkv, h, w.eps, pos, cos, sin, 0.5, bias=bias).double()
    t = torch.from_numpy(np.asarray(oracle.rmsnorm_linear(w.a, w.g, w.W, w.eps))).to(dev).double() + bias.double()
    p = t[:, : (Hq + Hkv) * h].reshape(M, -1, h // 2, 2)
    c, s = cos.double()[pos.long()][:, None], sin.double()[pos.long()][:, None]
    r = torch.stack((p[..., 0] * c - p[..., 1] * s, p[..., 0] * s + p[..., 1] * c), -1).flatten(1)
    r[:, : Hq * h] *= 0.5
    want = torch.cat((r, t[:, (Hq + Hkv) * h:]), 1)
    assert float(((y - want).abs().amax(1) / want.abs().amax(1)).max()) <= TOL


@pytest.mark.gpu
@pytest.mark.parametrize("M", [3, 40, 333])
def test_prefill_names_the_tile_kernel(M):
    # PREFILL forces the tile kernel at any M: the bits of its automatic tile here, 128 x 96.
    from paper_2407_09577_amd import flashnorm as fn
    K, N = 512, 3000
    w = workloads.make("linear", M, K, N, eps=1e-5, seed=M)
    Ws, _, _ = fn.fold_weights(w.W.cuda(), w.g.cuda())
    a, s = w.a.cuda(), torch.empty(M, device="cuda")
    y = fn.flashnorm_linear(a, Ws, N, w.eps, path=fn.FN_PATH_PREFILL)
    assert torch.equal(y, fn.flashnorm_linear(a, Ws, N, w.eps, path=fn.FN_PATH_PREFILL | (4 << 8)))
    # A kind that takes no named tile: the same products, unscaled (its sums in the tiles' one order over K).
    ones = torch.ones(M, device="cuda")
    z = fn.flashnorm_linear_relu(a, Ws, N, w.eps, s, path=fn.FN_PATH_PREFILL)
    assert torch.equal(z, fn.rowscale_linear(a, Ws, N, ones, path=fn.FN_PATH_PREFILL).clamp(min=0))


class _Call:
    """Seeded operands on the GPU (activations in rows padded with NaN), and fp64 products of them."""

    def __init__(self, M, K, N, glu, mean=0.0):
        gen = torch.Generator(device="cuda").manual_seed(M + K + N)
        a = (torch.randn(M, K, generator=gen, device="cuda") + mean).to(torch.bfloat16)
        big = torch.full((M, K + 24), float("nan"), dtype=torch.bfloat16, device="cuda")
        big[:, :K] = a
        self.a, self.g = big[:, :K], torch.rand(K, generator=gen, device="cuda") + 0.5
        self.W = (torch.randn(K, N, generator=gen, device="cuda") * K ** -0.5).to(torch.bfloat16)
        self.beta = torch.randn(K, generator=gen, device="cuda") * 0.3
        self.M, self.N, self.eps = M, N, 1e-5
        self.x = a.double()
        self.t = (self.x * self.g.double()) @ self.W.double()
        self.s = (self.eps + self.x.square().mean(1, keepdim=True)).rsqrt()
        self.layout = 1 if glu else 0
        self.inv = torch.full((M,), float("nan"), device="cuda")

    def pack(self, g=True, **kw):
        from paper_2407_09577_amd import flashnorm as fn
        return fn.fold_weights(self.W, self.g if g else None, layout=self.layout, **kw)

    def check_inv(self):
        assert float((self.inv.double() / self.s[:, 0] - 1).abs().max()) <= 1e-5


def _row_err(y, ref):
    assert y.shape == ref.shape and bool(torch.isfinite(y).all())
    return float(((y.double() - ref).abs().amax(1) / ref.abs().amax(1)).max())


def _rotate(v, pos, cos, sin):
    p = v.reshape(v.shape[0], -1, cos.shape[1], 2)
    c, s = cos.double()[pos.long()][:, None], sin.double()[pos.long()][:, None]
    return torch.stack((p[..., 0] * c - p[..., 1] * s, p[..., 0] * s + p[..., 1] * c), -1).flatten(1)


@pytest.mark.gpu
@pytest.mark.parametrize("shape,dims", [(s, d) for s, d, _ in SHAPE_CALLS if d])
def test_plain_kinds_on_every_shape(shape, dims):
    from paper_2407_09577_amd import flashnorm as fn
    M, K, N = dims
    assert _shape(M, K, N) == shape
    c = _Call(M, K, N, False)
    Ws = c.pack()[0]
    bias = torch.randn(N, device="cuda")
    assert _row_err(fn.flashnorm_linear(c.a, Ws, N, c.eps, bias=bias, inv_rms=c.inv), c.t * c.s + bias.double()) <= TOL
    c.check_inv()
    c.inv.fill_(float("nan"))
    assert _row_err(fn.flashnorm_linear_relu(c.a, Ws, N, c.eps, c.inv), c.t.clamp(min=0)) <= TOL
    c.check_inv()
    assert _row_err(fn.rowscale_linear(c.a, Ws, N, c.s[:, 0].float()), c.t * c.s) <= TOL
    assert _row_err(fn.baseline_rmsnorm_linear(c.a, c.g, c.pack(g=False)[0], N, c.eps), c.t * c.s) <= TOL
    c = _Call(M, K, N, False, mean=0.5)
    Wl, cs, cb = c.pack(beta=c.beta, colsum=True, c_star=True)
    d = c.x - c.x.mean(1, keepdim=True)
    d = d / (d.square().mean(1, keepdim=True) + c.eps).sqrt() * c.g.double() + c.beta.double()
    assert _row_err(fn.flashnorm_layernorm_linear(c.a, Wl, cs, cb, N, c.eps), d @ c.W.double()) <= TOL
    heads = N // 4
    c = _Call(M, K, 4 * heads, False)
    Hkv = heads // 5
    Hq = heads - 2 * Hkv
    cos, sin = (v.cuda() for v in workloads.rope_tables(64, 4))
    pos = torch.arange(M, device="cuda", dtype=torch.int32) % 64
    qk = (Hq + Hkv) * 4
    want = torch.cat((_rotate((c.t * c.s)[:, :qk], pos, cos, sin), (c.t * c.s)[:, qk:]), 1)
    want[:, : Hq * 4] *= 0.5
    y = fn.flashnorm_qkv_rope(c.a, c.pack()[0], Hq, Hkv, 4, c.eps, pos, cos, sin, 0.5, inv_rms=c.inv)
    assert _row_err(y, want) <= TOL
    c.check_inv()


@pytest.mark.gpu
@pytest.mark.parametrize("shape,dims", [(s, d) for s, _, d in SHAPE_CALLS if d])
def test_glu_kinds_on_every_shape(shape, dims):
    from paper_2407_09577_amd import flashnorm as fn
    M, K, N = dims
    F = N // 2
    assert _shape(M, K, N, True) == shape
    c = _Call(M, K, N, True)
    Wg = c.pack()[0]
    gate, up = c.t[:, :F], c.t[:, F:]
    silu = (gate * c.s) * torch.sigmoid(gate * c.s)
    assert _row_err(fn.flashnorm_glu(c.a, Wg, F, c.eps), silu * up * c.s) <= TOL
    assert _row_err(fn.flashnorm_glu_act(c.a, Wg, F, c.eps, fn.FN_GLU_REGLU), gate.clamp(min=0) * up * c.s ** 2) <= TOL
    assert _row_err(fn.flashnorm_glu_act(c.a, Wg, F, c.eps, fn.FN_GLU_BILINEAR), gate * up * c.s ** 2) <= TOL
    y = fn.flashnorm_glu_act(c.a, Wg, F, c.eps, fn.FN_GLU_SWIGLU_DEFER_UP, inv_rms=c.inv)
    assert _row_err(y, silu * up) <= TOL
    c.check_inv()
    assert _row_err(fn.baseline_rmsnorm_glu(c.a, c.g, c.pack(g=False)[0], F, c.eps), silu * up * c.s) <= TOL


@pytest.mark.gpu
@pytest.mark.parametrize("shape", [0, 7, 9, 12, 16, 17])
def test_nonfinite_rows_stay_in_their_row(shape):
    # Rows holding NaN or an infinity are NaN throughout (their mean square is not finite), every other row has the
    # bits it has beside finite rows.
    from paper_2407_09577_amd import flashnorm as fn
    for glu, dims in ((False, SHAPE_CALLS[shape][1]), (True, SHAPE_CALLS[shape][2])):
        if dims is None:
            continue
        M, K, N = dims
        c = _Call(M, K, N, glu, mean=0.25)
        bad = {1: float("nan"), 17: float("inf"), M - 1: float("-inf")}
        ruined = c.a.clone()
        for r, v in bad.items():
            ruined[r, (7 * r) % K] = v
        Ws, cs, cb = c.pack(beta=None if glu else c.beta, colsum=not glu, c_star=not glu)
        calls = [lambda a: fn.flashnorm_glu(a, Ws, N // 2, c.eps)] if glu else [
            lambda a: fn.flashnorm_linear(a, Ws, N, c.eps),
            lambda a: fn.flashnorm_layernorm_linear(a, Ws, cs, cb, N, c.eps)]
        good = torch.tensor([r not in bad for r in range(M)], device="cuda")
        for call in calls:
            clean, got = call(c.a), call(ruined)
            assert bool(torch.isnan(got[~good]).all())
            assert bool(torch.isfinite(clean).all()) and torch.equal(got[good], clean[good])
