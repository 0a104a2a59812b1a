"""Middle-row kernel (csrc/mid_kernel.h): its register use on the CPU, and on the GPU every kind at the
edges of its tiles (row blocks and groups, ragged columns and K, the smallest and the largest of its
range) against the fp64 oracle, with the row error bar of the other bf16 paths."""
import ctypes

import numpy as np
import pytest
import torch

import oracle
from _codeobj import kernel_resources
from paper_2407_09577_amd import workloads

TOL = 2e-2  # row-normwise, bf16: one rounding of W* and one of the output (2 x 2^-8) and the fp32 sums


@pytest.mark.parametrize("source", ["mid_kinds_a.hip", "mid_kinds_b.hip", "mid_kinds_c.hip"])
def test_no_spills(source, tmp_path):
    res = kernel_resources(source, tmp_path)
    assert res
    assert [n for n, f in res.items() if f.get("private_segment_fixed_size", 0) or f.get("vgpr_spill_count", 0)] == []


def _shape(M, K, N, glu=False):
    """The workgroup shape that the built library takes for a call (-1: the tile kernel)."""
    from paper_2407_09577_amd import flashnorm as fn
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
