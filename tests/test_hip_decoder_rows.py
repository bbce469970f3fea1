"""Row kernels of the training step (csrc/decoder.hip) against fp64 on the CPU."""
import ctypes as C

import pytest
import torch

import paper_2505_16710_amd as seco

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
F32, BF16 = 0, 1
U = 2.0 ** -24            # half an ulp of fp32, relative


def _call(name, *args):
    """dec_<name>: tensors by address, Python integers as int64 (the first one, the dtype, as int), then the stream."""
    fn = getattr(seco.load_library(), "dec_" + name)
    conv = [C.c_int(args[0])]
    for a in args[1:]:
        conv.append(C.c_void_p(None if a is None else a.data_ptr()) if a is None or torch.is_tensor(a) else C.c_int64(a))
    assert fn(*conv, C.c_void_p(torch.cuda.current_stream().cuda_stream)) == 0
    torch.cuda.synchronize()


def _silu64(u):
    s = torch.sigmoid(u)
    return u * s, s


def test_silu_in_fp32_keeps_fp32_precision():
    """exp, 3 ulp at most, one addition, one division and one or three products behind it: below 10 U, at arguments where
    an exponential whose argument is scaled in fp32 is off by |x| U."""
    u = torch.linspace(-80, 80, 40001)
    u64, dev = u.double(), u.to(DEV)
    out = torch.empty_like(dev)
    _call("silu", F32, dev, out, u.numel())
    ref, s = _silu64(u64)
    assert float(((out.cpu().double() - ref).abs() / ref.abs().clamp_min(1e-300))[ref != 0].max()) < 10 * U
    g = torch.randn(u.numel(), generator=torch.Generator().manual_seed(1))
    d = g.to(DEV)
    _call("silu_bwd", F32, dev, d, u.numel())
    ref = g.double() * s * (1 + u64 * torch.sigmoid(-u64))
    scale = g.double().abs() * s * (1 + u64.abs() * torch.sigmoid(-u64))
    # 1 - s of an s that is within 6 U of its value
    scale = scale + g.double().abs() * s * u64.abs() * s
    assert float(((d.cpu().double() - ref).abs() / scale).max()) < 14 * U


@pytest.mark.parametrize("v", [29, 1000])
def test_cross_entropy_in_fp32_keeps_fp32_precision(v):
    """Logits that are multiples of 2^-10 within 64 of each other: their differences are exact, so that a probability is off
    by the exponential (3 ulp), the sum (its partial sums) and two products."""
    rows = 37
    gen = torch.Generator().manual_seed(v)
    logits = torch.randint(-32 * 1024, 32 * 1024, (rows, v), generator=gen).float() / 1024
    target = torch.randint(0, v, (rows,), generator=gen)
    dev, loss = logits.to(DEV), torch.empty(rows, device=DEV)
    _call("cross_entropy", F32, dev, target.to(DEV), loss, rows, v)
    lse = torch.logsumexp(logits.double(), 1)
    ref = lse - logits.double().gather(1, target[:, None])[:, 0]
    assert float((loss.cpu().double() - ref).abs().max()) < 64 * 8 * U
    _call("cross_entropy", F32, dev, target.to(DEV), None, rows, v)
    p = torch.exp(logits.double() - lse[:, None])
    off = torch.ones_like(p).scatter_(1, target[:, None], 0.0).bool()
    assert float(((dev.cpu().double() - p).abs() / p)[off].max()) < 24 * U
    on = dev.cpu().double().gather(1, target[:, None]) - (p.gather(1, target[:, None]) - 1)
    assert float(on.abs().max()) < 24 * U


@pytest.mark.parametrize("dtype", [F32, BF16])
@pytest.mark.parametrize("rows,d,v,kind", [
    (1, 8, 1, "uniform"), (300, 64, 29, "uniform"), (257, 29, 5, "uniform"), (64, 2056, 7, "negative"),
    (2049, 40, 3, "same"), (2500, 1032, 1000, "same"), (4500, 16, 900, "frequent"), (2048, 1027, 2, "frequent"),
])
def test_embedding_gradient(dtype, rows, d, v, kind):
    """Rows of a token are added in fp32, in order: within (n + 1) U of the sum of their magnitudes, and one rounding."""
    gen = torch.Generator().manual_seed(rows + d)
    dt = torch.float32 if dtype == F32 else torch.bfloat16
    x = torch.randn(rows, d, generator=gen).to(dt)
    base = torch.randn(v + 1, d, generator=gen).to(dt)          # the last row lies behind the table
    tok = torch.randint(0, v, (rows,), generator=gen)
    if kind == "negative":
        tok = torch.where(torch.rand(rows, generator=gen) < 0.5, tok - v, tok)
    elif kind == "same":
        tok[:] = v - 1
    elif kind == "frequent":
        tok[torch.rand(rows, generator=gen) < 0.4] = 0
    grad = base.to(DEV)
    _call("embedding_bwd", dtype, x.to(DEV), tok.to(DEV), grad, rows, d, v)
    at = torch.where(tok < 0, tok + v, tok)
    ref = base.double().index_add(0, at, x.double())
    size = base.double().abs().index_add(0, at, x.double().abs())
    n = torch.bincount(at, minlength=v + 1)[:, None].double()
    bound = (n + 1) * U * size + (2.0 ** -8 * ref.abs() if dtype == BF16 else 0)
    assert torch.equal(grad[v].cpu(), base[v])
    assert ((grad.cpu().double() - ref).abs() <= bound).all()
