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


# Row lengths: the blocks of a row kept in registers are 1, 2 or 4 of 256 words (a word: 8 bf16 or 4 fp32 where the rows
# start on 16-byte boundaries, else one element), what is left of a longer row is read twice.
LENGTHS = [(BF16, 8), (BF16, 2048), (BF16, 2056), (BF16, 4096), (BF16, 4104), (BF16, 8192), (BF16, 10248),
           (F32, 4), (F32, 1024), (F32, 1028), (F32, 2052), (F32, 4096), (F32, 5000),
           (BF16, 1), (BF16, 255), (BF16, 257), (BF16, 513), (BF16, 1025), (F32, 1023), (F32, 2047)]


def _rows(dtype, seed, *shape):
    x = torch.randn(*shape, generator=torch.Generator().manual_seed(seed))
    return x.to(torch.float32 if dtype == F32 else torch.bfloat16)


def _norm64(x, gain):
    r = torch.rsqrt((x * x).mean(1, keepdim=True) + 1e-6)
    return r, x * r, x * r * gain


@pytest.mark.parametrize("residual", ["none", "in place", "apart"])
@pytest.mark.parametrize("dtype,d", LENGTHS)
def test_add_rmsnorm(dtype, d, residual):
    """Sums of d squares and a reciprocal root in fp32 (64 U), then a rounding of the row and one of the product."""
    rows = 5
    x, y, gain = _rows(dtype, d, rows, d), _rows(dtype, d + 1, rows, d), _rows(dtype, d + 2, d) + 1
    dx, dy = x.to(DEV), None if residual == "none" else y.to(DEV)
    out = None if residual == "none" else dx if residual == "in place" else torch.empty_like(dx)
    h, r = torch.empty_like(dx), torch.empty(rows, device=DEV)
    _call("add_rmsnorm", dtype, dx, dy, gain.to(DEV), out, h, r, rows, d)
    s = x if dy is None else (x.float() + y.float()).to(x.dtype)
    if out is not None:
        assert torch.equal(out.cpu(), s)
    if residual != "in place":
        assert torch.equal(dx.cpu(), x)
    r64, _, h64 = _norm64(s.double(), gain.double())
    eps = 64 * U + (2.0 ** -7 + 2.0 ** -16 if dtype == BF16 else 0)     # (two roundings to 8 bits, 2^-8 each)
    assert ((r.cpu().double()[:, None] - r64).abs() <= 64 * U * r64).all()
    assert ((h.cpu().double() - h64).abs() <= eps * h64.abs()).all()


@pytest.mark.parametrize("rows,d_in", [(1, "none"), (7, "in place"), (300, "apart"), (300, "none")])
@pytest.mark.parametrize("dtype,d", LENGTHS)
def test_rmsnorm_backward(dtype, d, rows, d_in):
    """Terms and sums in fp32, 64 U of the magnitudes added up; in bf16 one rounding of d_x, and the normalised row of the
    gain's gradient rounded first."""
    x, dh, extra = (_rows(dtype, d + i, rows, d) for i in (3, 4, 5))
    gain, r = _rows(dtype, d + 6, d) + 1, None
    r64, n64, _ = _norm64(x.double(), gain.double())
    r = r64[:, 0].float()
    n64 = x.double() * r.double()[:, None]
    part = torch.randn(256, d, generator=torch.Generator().manual_seed(d + 7))
    dev = {"x": x.to(DEV), "dh": dh.to(DEV), "in": extra.to(DEV), "part": part.to(DEV)}
    out = dev["in"] if d_in == "in place" else torch.empty_like(dev["x"])
    _call("rmsnorm_bwd", dtype, dev["x"], gain.to(DEV), r.to(DEV), dev["dh"], None if d_in == "none" else dev["in"], out,
          dev["part"], rows, d)
    e = dh.double() * gain.double()
    mean, mean_abs = (e * n64).mean(1, keepdim=True), (e * n64).abs().mean(1, keepdim=True)
    base = torch.zeros_like(e) if d_in == "none" else extra.double()
    r64 = r.double()[:, None]
    ref = base + r64 * (e - n64 * mean)
    size = base.abs() + r64 * (e.abs() + n64.abs() * mean_abs)
    eps = 2.0 ** -8 if dtype == BF16 else 0.0
    assert ((out.cpu().double() - ref).abs() <= 64 * U * size + eps * ref.abs()).all()
    got = dev["part"].cpu().double().sum(0) - part.double().sum(0)
    want = (dh.double() * n64).sum(0)
    size = part.double().abs().sum(0) + (dh.double() * n64).abs().sum(0)
    assert ((got - want).abs() <= 64 * U * size + eps * (dh.double() * n64).abs().sum(0)).all()
    if rows < 256:
        assert torch.equal(dev["part"].cpu()[rows:], part[rows:])


@pytest.mark.parametrize("dtype,d", [(F32, 64), (F32, 260), (F32, 512), (F32, 516), (F32, 1024), (F32, 131), (F32, 1028),
                                     (BF16, 512), (BF16, 520), (BF16, 1024), (BF16, 1032), (BF16, 2048), (BF16, 255), (BF16, 2056)])
@pytest.mark.parametrize("rows,d_in", [(257, "in place"), (513, "apart"), (1030, "in place")])
def test_rmsnorm_backward_with_a_wavefront_per_row(dtype, d, rows, d_in):
    """Both sides of its lengths (64, 128 and 256 words) and of its rows; a last round in which wavefronts have none."""
    test_rmsnorm_backward(dtype, d, rows, d_in)


@pytest.mark.parametrize("dtype", [F32, BF16])
@pytest.mark.parametrize("v", [1, 29, 2048, 4104, 10000])
def test_cross_entropy_targets(dtype, v):
    """Targets inside, -100 (no loss, no gradient) and outside (NaN in that row alone)."""
    rows = 8
    logits = 4 * _rows(dtype, v, rows, v).float()
    logits = logits.to(torch.float32 if dtype == F32 else torch.bfloat16)
    target = torch.randint(0, v, (rows,), generator=torch.Generator().manual_seed(v))
    target[1], target[3], target[4], target[6] = -100, v, -1, v - 1
    dev, loss = logits.to(DEV), torch.empty(rows, device=DEV)
    _call("cross_entropy", dtype, dev, target.to(DEV), loss, rows, v)
    assert torch.equal(dev.cpu(), logits)
    good = torch.tensor([0, 2, 5, 6, 7])
    lse = torch.logsumexp(logits.double(), 1)
    ref = lse[good] - logits.double()[good, target[good]]
    assert float((loss.cpu().double()[good] - ref).abs().max()) < 64 * U * max(1.0, float(lse.abs().max()))
    assert float(loss[1]) == 0.0 and torch.isnan(loss[3:5]).all()
    _call("cross_entropy", dtype, dev, target.to(DEV), None, rows, v)
    got = dev.cpu().double()
    p = torch.softmax(logits.double(), 1)
    ref = p.clone()
    ref[good, target[good]] -= 1
    eps = 256 * U + (2.0 ** -8 if dtype == BF16 else 0)                 # bf16 rows: exp is off by |x| U, |x| < 64
    assert ((got - ref)[good].abs() <= eps * (ref[good].abs() + 256 * U)).all()
    assert not got[1].any() and torch.isnan(got[3:5]).all()


@pytest.mark.parametrize("dtype", [F32, BF16])
@pytest.mark.parametrize("v", [1, 29, 2048, 10000])
def test_cross_entropy_loss_and_gradient_in_one_launch(dtype, v):
    """The same bits as the two calls, whichever thread holds the target."""
    rows = 300
    logits = 4 * _rows(dtype, v, rows, v).float()
    logits = logits.to(torch.float32 if dtype == F32 else torch.bfloat16).to(DEV)
    target = torch.randint(0, v, (rows,), generator=torch.Generator().manual_seed(v)).to(DEV)
    target[1], target[3], target[4], target[6], target[7] = -100, v, -1, v - 1, 0
    one, two, loss1, loss2 = logits.clone(), logits.clone(), torch.empty(rows, device=DEV), torch.empty(rows, device=DEV)
    _call("cross_entropy", dtype, one, target, loss1, rows, v)
    _call("cross_entropy", dtype, one, target, None, rows, v)
    _call("cross_entropy_both", dtype, two, target, loss2, rows, v)
    bits = torch.int32 if dtype == F32 else torch.int16
    assert torch.equal(one.view(bits), two.view(bits)) and torch.equal(loss1.view(torch.int32), loss2.view(torch.int32))


@pytest.mark.parametrize("dtype,n", [(BF16, 8), (BF16, 9), (BF16, 65536 * 2048 + 2048 * 3), (F32, 4), (F32, 1023)])
def test_silu_lengths(dtype, n):
    """The shortest and odd lengths, and one that the largest grid walks more than once."""
    u = _rows(dtype, 1, min(n, 1 << 20)).repeat(-(-n // (1 << 20)))[:n].contiguous()
    dev = u.to(DEV)
    out = torch.zeros(n + 8, dtype=u.dtype, device=DEV)
    _call("silu", dtype, dev, out, n)
    assert not out[n:].any()
    f = dev.float()
    ref = f * torch.sigmoid(f)
    eps = 16 * U + (2.0 ** -8 if dtype == BF16 else 0)
    assert ((out[:n].float() - ref).abs() <= eps * ref.abs()).all()


@pytest.mark.parametrize("dtype,B,Hq,Hkv,n,D,row0", [
    (BF16, 1, 8, 2, 512, 128, 1024), (BF16, 2, 3, 1, 17, 128, 0), (BF16, 1, 9, 9, 1, 128, 5),
    (F32, 2, 3, 1, 17, 128, 0), (F32, 2, 5, 5, 33, 80, 7), (F32, 1, 4, 4, 1, 8, 3), (F32, 1, 6, 3, 40, 256, 100),
])
def test_rotated_projection_in_one_launch(dtype, B, Hq, Hkv, n, D, row0):
    """dec_rope_qkv against the public calls it stands for: the same bits, and nothing else of the cache is written."""
    base, N, dt = 500000.0, row0 + n + 5, torch.bfloat16 if dtype == BF16 else torch.float32
    gen = torch.Generator(device=DEV).manual_seed(n + D)
    qkv = torch.randn(B, n, Hq + 2 * Hkv, D, generator=gen, device=DEV).to(dt)
    k, v = (torch.randn(B, Hkv, N, D, generator=gen, device=DEV).to(dt) for _ in range(2))
    gk, gv = (torch.randn(B, Hkv, N, D, generator=gen, device=DEV) for _ in range(2))

    def parts(x):
        x = x.transpose(1, 2)
        return x[:, :Hq], x[:, Hq:Hq + Hkv], x[:, Hq + Hkv:]

    def call(inverse, t, kk, vv):
        fn = seco.load_library().dec_rope_qkv
        st = (C.c_int64 * 3)(*kk.stride()[:3])
        rc = fn(dtype, inverse, C.c_void_p(t.data_ptr()), C.c_void_p(kk.data_ptr()), C.c_void_p(vv.data_ptr()), st,
                *(C.c_int64(x) for x in (B, Hq, Hkv, n, D, row0)), C.c_float(base), C.c_void_p(torch.cuda.current_stream().cuda_stream))
        assert rc == 0
        torch.cuda.synchronize()
    x, kk, vv = qkv.clone(), k.clone(), v.clone()
    call(0, x, kk, vv)
    q, kn, vn = parts(qkv)
    want_k, want_v = k.clone(), v.clone()
    seco.kv_append(kn.contiguous(), vn.contiguous(), want_k, want_v, row0, rope_base=base)
    assert torch.equal(kk, want_k) and torch.equal(vv, want_v)
    assert torch.equal(parts(x)[0], seco.rope_rotate(q.contiguous(), row0, base))
    assert torch.equal(x[:, :, Hq:], qkv[:, :, Hq:])
    x, kk, vv = qkv.clone(), gk.clone(), gv.clone()
    call(1, x, kk, vv)
    dk, dv = seco.kvgrad_readout(gk, gv, row0, n, dt, rope_base=base)
    assert torch.equal(parts(x)[0], seco.rope_rotate(q.contiguous(), row0, base, inverse=True))
    assert torch.equal(parts(x)[1], dk) and torch.equal(parts(x)[2], dv) and torch.equal(kk, gk) and torch.equal(vv, gv)


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("d", [8, 200, 1024, 1031, 2056, 8208])
def test_norm_of_embedded_rows(dtype, d):
    """dec_embed_rmsnorm against the gathered rows through dec_add_rmsnorm: the same bits.  Row lengths of one, two and four kept
    blocks and beyond, with and without 16-byte accesses; negative tokens; tokens outside the table give NaN rows and no others."""
    code, v, rows = (F32 if dtype == torch.float32 else BF16), 11, 37
    g = torch.Generator().manual_seed(d)
    table, gain = torch.randn(v, d, generator=g).to(dtype).to(DEV), torch.randn(d, generator=g).to(dtype).to(DEV)
    token = torch.randint(-v, v, (rows,), generator=g).to(DEV)
    new = lambda: (torch.empty(rows, d, dtype=dtype, device=DEV), torch.empty(rows, d, dtype=dtype, device=DEV), torch.empty(rows, device=DEV))
    x = table[token]
    _, h_ref, r_ref = new()
    _call("add_rmsnorm", code, x, None, gain, None, h_ref, r_ref, rows, d)
    x_out, h, r = new()
    _call("embed_rmsnorm", code, table, token, gain, x_out, h, r, rows, d, v)
    assert torch.equal(x_out, x) and torch.equal(h, h_ref) and torch.equal(r, r_ref)
    token[3], token[20] = v, -v - 1
    _call("embed_rmsnorm", code, table, token, gain, x_out, h, r, rows, d, v)
    bad = torch.zeros(rows, dtype=torch.bool, device=DEV)
    bad[[3, 20]] = True
    assert x_out[bad].isnan().all() and h[bad].isnan().all()
    assert torch.equal(x_out[~bad], x[~bad]) and torch.equal(h[~bad], h_ref[~bad])


@pytest.mark.parametrize("n,d", [(1, 1), (3, 64), (5, 1000), (2, 65)])
def test_sums_of_the_gains_parts(n, d):
    """256 terms: fp32 additions in chains of at most 31, so below 31 U of the sum of magnitudes; the rounded one is its rounding."""
    parts = torch.randn(n, 256, d, generator=torch.Generator().manual_seed(d))
    sums = torch.empty(n, d, device=DEV)
    for code, dtype in ((F32, torch.float32), (BF16, torch.bfloat16)):
        rounded = torch.empty(n, d, dtype=dtype, device=DEV)
        _call("gain_sums", code, parts.to(DEV), sums, rounded, n, d)
        ref, scale = parts.double().sum(1), parts.double().abs().sum(1)
        assert float(((sums.cpu().double() - ref).abs() / scale).max()) < 31 * U
        assert torch.equal(rounded, sums.to(dtype))


@pytest.mark.parametrize("rows,widths", [(1, (16, 16, 16)), (37, (2048, 512, 512)), (300, (48, 16, 96))])
def test_runs_of_columns_to_matrices_of_their_own(rows, widths):
    src = torch.randint(0, 256, (rows, sum(widths)), dtype=torch.uint8, device=DEV)
    out = [torch.empty(rows, w, dtype=torch.uint8, device=DEV) for w in widths]
    fn = seco.load_library().dec_split_columns
    P, I = C.c_void_p, C.c_int64
    fn.argtypes = [P] * 4 + [I] * 4 + [P]
    assert fn(src.data_ptr(), *(t.data_ptr() for t in out), rows, *widths, torch.cuda.current_stream().cuda_stream) == 0
    for t, ref in zip(out, src.split(widths, 1)):
        assert torch.equal(t, ref)
    assert fn(src.data_ptr(), *(t.data_ptr() for t in out), rows, 24, 16, 16, torch.cuda.current_stream().cuda_stream) != 0


@pytest.mark.parametrize("B,Hq,Hkv,n,K,row0", [
    (1, 1, 1, 1, 64, 0), (2, 3, 1, 17, 192, 5), (1, 9, 9, 33, 128, 30000),        # tiles of 32 x 64, half of a head
    (1, 8, 2, 512, 1024, 1024), (2, 8, 2, 201, 128, 3),                           # 64 x 64
    (1, 8, 2, 1000, 192, 7), (3, 8, 2, 333, 64, 0),                               # 64 x 128, a whole head
    (1, 8, 2, 1000, 2048, 1), (1, 8, 2, 2048, 64, 9),                             # 128 rows: in two launches
])
def test_projection_rotated_in_its_product(B, Hq, Hkv, n, K, row0):
    """dec_gemm_qkv against dec_gemm and dec_rope_qkv: the same bits of queries and cache, and nothing else of the cache is written."""
    base, N, W = 500000.0, row0 + n + 5, (Hq + 2 * Hkv) * 128
    gen = torch.Generator(device=DEV).manual_seed(n + K)
    h, w = (torch.randn(*s, generator=gen, device=DEV).to(torch.bfloat16) for s in ((B * n, K), (K, W)))
    k, v = (torch.randn(B, N, Hkv, 128, generator=gen, device=DEV).to(torch.bfloat16).transpose(1, 2) for _ in range(2))
    lib, s, p = seco.load_library(), C.c_void_p(torch.cuda.current_stream().cuda_stream), lambda t: C.c_void_p(t.data_ptr())
    i64, st = lambda *x: [C.c_int64(y) for y in x], (C.c_int64 * 3)(*k.stride()[:3])
    want, wk, wv = torch.empty(B * n, W, dtype=torch.bfloat16, device=DEV), k.clone(), v.clone()
    assert wk.stride() == k.stride()
    assert lib.dec_gemm(0, 0, p(h), p(w), p(want), None, *i64(B * n, W, K, K, W, W), s) == 0
    assert lib.dec_rope_qkv(BF16, 0, p(want), p(wk), p(wv), st, *i64(B, Hq, Hkv, n, 128, row0), C.c_float(base), s) == 0
    got = torch.empty_like(want)
    assert lib.dec_gemm_qkv(p(h), p(w), p(got), p(k), p(v), st, *i64(B, Hq, Hkv, n, K, row0), C.c_float(base), s) == 0
    torch.cuda.synchronize()
    assert torch.equal(got[:, :Hq * 128], want[:, :Hq * 128]) and torch.equal(k, wk) and torch.equal(v, wv)
