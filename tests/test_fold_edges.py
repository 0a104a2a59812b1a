"""fold_weights at the values and views where its rounding or its loads can go wrong: products that tie,
underflow, overflow or are not finite, K and N off the 16-byte runs, unaligned views, both source and
storage types, against fp64 products rounded once on the CPU, bit for bit."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


def _bf16_bits(x):
    """fp64 -> bf16 bits, nearest even (7 explicit bits; fixed spacing 2^-133 below 2^-126)."""
    x = np.asarray(x, dtype=np.float64)
    with np.errstate(all="ignore"):
        m, e = np.frexp(x)
        q = np.maximum(e - 8, -133)
        y = np.ldexp(np.rint(np.ldexp(x, -q)), q)
        y = np.where(np.isfinite(x) & (np.abs(y) > 3.3895313892515355e38), np.copysign(np.inf, x), y)
        y = np.where(np.isfinite(x), y, x).astype(np.float32)
    bits = (y.view(np.uint32) >> 16).astype(np.uint16)
    return np.where(np.isnan(x), np.uint16(0x7FC0), bits)


def _values(K, N, dtype, seed):
    gen = torch.Generator().manual_seed(seed)
    W = torch.randn(K, N, generator=gen)
    W *= torch.exp2(torch.randint(-140, 120, (K, N), generator=gen).float() * (torch.rand(K, N, generator=gen) < 0.3))
    g = torch.rand(K, generator=gen) + 0.5
    g[::3] = torch.exp2(torch.randint(-20, 20, (len(g[::3]),), generator=gen).float())
    g[1::7] = (torch.randint(1, 256, (len(g[1::7]),), generator=gen) * 2 + 1) / 512.0  # ties with 8-bit weights
    W.view(-1)[5:: 97] = float("inf")
    W.view(-1)[11:: 131] = float("nan")
    W.view(-1)[17:: 61] = -0.0
    W.view(-1)[23:: 89] = 3.3e38
    return W.to(dtype), g


def _views(W):
    K, N = W.shape
    yield "rows", W.cuda()
    yield "transposed", W.t().contiguous().cuda().t()
    odd = torch.zeros(N, K + 3, dtype=W.dtype, device="cuda")  # rows of [N, K] off the 16-byte runs
    odd[:, 1:K + 1] = W.t().cuda()
    yield "offset", odd[:, 1:K + 1].t()


@pytest.mark.parametrize("src", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("ws", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("K,N,layout", [(8, 16, 0), (72, 33, 0), (520, 70, 0), (200, 2 * 24, 1), (1032, 2 * 37, 1)])
def test_fold_bits(src, ws, K, N, layout):
    from paper_2407_09577_amd import flashnorm as fn
    W, g = _values(K, N, src, K + N)
    code = fn.FN_BF16 if ws == torch.bfloat16 else fn.FN_F32
    for use_g in (True, False):
        with np.errstate(all="ignore"):
            want = (g.double() if use_g else torch.ones(K).double())[:, None].numpy() * W.double().numpy()
            want_bits = _bf16_bits(want) if ws == torch.bfloat16 else want.astype(np.float32).view(np.uint32)
        for name, view in _views(W):
            Ws, _, _ = fn.fold_weights(view, g.cuda() if use_g else None, layout=layout, ws_dtype=ws)
            got = fn.unpack_weights(Ws, K, N, layout, code).cpu()
            got = got.view(torch.int16 if ws == torch.bfloat16 else torch.int32).numpy().view(want_bits.dtype)
            if ws == torch.float32:  # which NaN is the arithmetic's choice
                nan = np.isnan(want)
                assert np.isnan(got.view(np.float32)[nan]).all()
                got, expect = np.where(nan, 0, got), np.where(nan, 0, want_bits)
            else:
                expect = want_bits
            np.testing.assert_array_equal(got, expect, err_msg=f"{name} g={use_g}")


@pytest.mark.parametrize("src,ws", [(torch.bfloat16, torch.bfloat16), (torch.float32, torch.bfloat16),
                                    (torch.float32, torch.float32)])
@pytest.mark.parametrize("K,N", [(8, 5), (72, 33), (1000, 16), (4160, 130)])
def test_sums_follow_the_stored_values(src, ws, K, N):
    from paper_2407_09577_amd import flashnorm as fn
    gen = torch.Generator().manual_seed(K)
    W = (torch.randn(K, N, generator=gen) * K ** -0.5).to(src)
    g, beta = torch.rand(K, generator=gen) + 0.5, torch.randn(K, generator=gen)
    ref = None
    for name, view in _views(W):
        Ws, cs, cb = fn.fold_weights(view, g.cuda(), beta=beta.cuda(), colsum=True, c_star=True, ws_dtype=ws)
        stored = fn.unpack_weights(Ws, K, N, 0, fn.FN_BF16 if ws == torch.bfloat16 else fn.FN_F32).cpu().double()
        for got, want in ((cs, stored.sum(0)), (cb, beta.double() @ W.double())):
            # rounded once to fp32; the fp64 sums are off by no more than K 2^-53 of the sum of magnitudes
            slack = 2 ** -24 * want.abs() + K * 2 ** -52 * stored.abs().sum(0).clamp(min=1)
            assert bool(((got.cpu().double() - want).abs() <= slack).all()), name
        only, none, _ = fn.fold_weights(view, g.cuda(), ws_dtype=ws)
        assert none is None and torch.equal(only, Ws), name
        if ref is not None:
            assert all(torch.equal(a, b) for a, b in zip(ref, (Ws, cs, cb))), name
        ref = (Ws, cs, cb)


@pytest.mark.parametrize("ws", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("K,N,sums", [(72, 33, False), (520, 70, False), (200, 5, True)])
def test_padding_is_positive_zero(ws, K, N, sums):
    """Rows past K and columns past N are +0 in every byte, whatever g holds (negative, infinite, NaN)."""
    from paper_2407_09577_amd import flashnorm as fn
    W, g = _values(K, N, ws, K)
    g[0], g[1], g[2::2] = float("nan"), float("-inf"), -1.0
    for name, view in _views(W):
        Ws, _, _ = fn.fold_weights(view, g.cuda(), colsum=sums, ws_dtype=ws)
        KP = (K + 63) // 64 * 64
        if ws == torch.bfloat16:  # [k block][column block][k chunk][column][8 k]
            bits = Ws.flatten().view(torch.int16)
            bits = bits.view(KP // 32, -1, 4, 16, 8).permute(0, 2, 4, 1, 3).reshape(KP, -1)
        else:
            bits = Ws.flatten().view(torch.int32).view(KP, -1)
        assert bits.shape[1] >= N
        assert not bits[K:].any() and not bits[:, N:].any(), name
        assert bits[:K, :N].any(), name


@pytest.mark.parametrize("src,ws", [(torch.bfloat16, torch.bfloat16), (torch.float32, torch.bfloat16),
                                    (torch.float32, torch.float32), (torch.bfloat16, torch.float32)])
@pytest.mark.parametrize("K,N,transposed", [(4160, 2000, True), (200, 72, False)])
def test_sums_over_the_inputs(src, ws, K, N, transposed):
    """colsum and c_star may take g's memory, and colsum alone W's: both are read before they are written."""
    from paper_2407_09577_amd import flashnorm as fn
    gen = torch.Generator().manual_seed(K)
    W = (torch.randn(K, N, generator=gen) * K ** -0.5).to(src).cuda()
    W = W.t().contiguous().t() if transposed else W
    g, beta = (torch.rand(K, generator=gen) + 0.5).cuda(), torch.randn(K, generator=gen).cuda()
    Ws, cs, cb = fn.fold_weights(W, g, beta=beta, colsum=True, c_star=True, ws_dtype=ws)

    def fold(W_, g_, colsum, c_star):
        out = torch.empty_like(Ws)
        rc = fn.lib().fold_weights(W_.data_ptr(), W_.stride(0), W_.stride(1), fn._dt(W_), g_.data_ptr(), beta.data_ptr(),
                                   K, N, fn.FN_LAYOUT_LINEAR, out.data_ptr(),
                                   fn.FN_BF16 if ws == torch.bfloat16 else fn.FN_F32, colsum, c_star,
                                   torch.cuda.current_stream().cuda_stream)
        assert rc == 0
        return out

    over = g.clone()
    assert torch.equal(fold(W, over, over.data_ptr(), over.data_ptr() + 4 * N), Ws)
    assert torch.equal(over[:N], cs) and torch.equal(over[N:2 * N], cb)
    over = g.clone()
    assert torch.equal(fold(W, over, None, over.data_ptr()), Ws) and torch.equal(over[:N], cb)
    # colsum over W
    mem = W.t().contiguous() if transposed else W.clone()
    view = mem.t() if transposed else mem
    assert torch.equal(fold(view, g, mem.data_ptr(), None), Ws)
    assert torch.equal(mem.flatten().view(torch.uint8)[: 4 * N].view(torch.float32), cs)
