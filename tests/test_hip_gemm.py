"""The decoder's matrix products (dec_gemm) against fp32 products of the same bf16 operands: every form and epilogue at the
edges of the tiles (64 and 128), of the contraction step (64) and of each shape of workgroup the launcher picks."""
import ctypes as C

import pytest
import torch

import paper_2505_16710_amd as seco

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
NN, NT, TN = 0, 1, 2
STORE, ADD, SILU, SILU_BWD = 0, 1, 2, 3


@pytest.mark.parametrize("form,epi,M,N,K", [
    (NN, STORE, 1, 8, 64), (NN, STORE, 63, 72, 64), (NN, STORE, 65, 136, 192), (NN, SILU, 129, 200, 320),
    (NT, STORE, 127, 64, 128), (NT, SILU_BWD, 130, 264, 448),
    (TN, STORE, 72, 200, 1), (TN, ADD, 136, 264, 77), (TN, ADD, 64, 64, 63), (TN, STORE, 128, 128, 129),
    # the contraction divided among the wavefronts of 32 x 64 tiles: fewer steps than wavefronts, one more, all in one round
    (NN, STORE, 31, 64, 448), (NN, SILU, 33, 72, 576), (NN, STORE, 500, 1024, 4096), (NT, STORE, 32, 8, 512),
    (NT, SILU_BWD, 65, 128, 640), (NT, STORE, 512, 1024, 1536),
    (NN, STORE, 640, 1024, 320), (NT, SILU_BWD, 700, 1000, 512),   # 64 x 64 tiles that fit one round, 32 x 64 do not
    (NN, STORE, 300, 4096, 64),            # more 64 x 64 tiles than CUs, two slots
    (NT, STORE, 1500, 1032, 2112),         # 128 x 64 tiles
    (NN, STORE, 1500, 1032, 2112), (NN, SILU, 2048, 1024, 2048),   # ... the steps halved between wavefronts, an odd number of them
    (TN, ADD, 2040, 2056, 200),            # 128 x 128 tiles, two groups, a remainder of the contraction
    (NN, SILU, 2050, 4104, 128),           # 128 x 128 tiles, one group, two workgroups per CU
    (NN, SILU, 500, 4000, 192), (TN, ADD, 1000, 1544, 200), (TN, STORE, 1000, 1544, 128),   # 64 x 128 tiles
    (NT, SILU_BWD, 1030, 4104, 128),       # 128 x 128 tiles, side by side: u requested early
    (TN, ADD, 2040, 2056, 40), (TN, ADD, 2040, 2056, 64),   # ... no whole step, one
])
def test_gemm_forms_and_epilogues(form, epi, M, N, K):
    lib = seco.load_library()
    P, I = C.c_void_p, C.c_int64
    lib.dec_gemm.argtypes = [C.c_int, C.c_int, P, P, P, P] + [I] * 6 + [P]
    g = torch.Generator(device=DEV).manual_seed(M + N + K)

    def normal(*shape):
        return torch.randn(*shape, generator=g, device=DEV).to(torch.bfloat16)
    a = normal(K, M) if form == TN else normal(M, K)
    b = normal(N, K) if form == NT else normal(K, N)
    c, c2 = normal(M + 1, N), normal(M + 1, N)                      # the last row must stay as it is
    c_in, c2_in = c.clone(), c2.clone()
    rc = lib.dec_gemm(form, epi, a.data_ptr(), b.data_ptr(), c.data_ptr(), c2.data_ptr(), M, N, K, a.shape[1], b.shape[1], N,
                      torch.cuda.current_stream().cuda_stream)
    assert rc == 0
    torch.cuda.synchronize()
    ref = torch.mm((a.float().t() if form == TN else a.float()).contiguous(), (b.float().t() if form == NT else b.float()).contiguous())
    if epi == ADD:
        ref += c_in[:M].float()
    if epi == SILU_BWD:
        u = c2_in[:M].float()
        s = torch.sigmoid(u)
        ref *= s * (1 + u * (1 - s))

    def close(x, y):
        return float((x.float() - y).abs().max() / y.abs().max()) < 1e-2 and float((x.float() - y).norm() / y.norm()) < 4e-3
    assert close(c[:M], ref)
    if epi == SILU:
        assert close(c2[:M], torch.nn.functional.silu(c[:M].float()))
    else:
        assert torch.equal(c2, c2_in)
    assert torch.equal(c[M], c_in[M]) and torch.equal(c2[M], c2_in[M])


@pytest.mark.parametrize("form,epi,M,N,K", [
    (TN, ADD, 4096, 1024, 72), (TN, STORE, 4088, 1032, 64),   # 128 x 128 tiles in four by two parts; in eight by one, the last tiles short
    (NN, STORE, 2048, 1032, 2112), (NT, STORE, 2040, 1024, 192),   # 128 x 64 and 64 x 64 tiles
    (NN, SILU, 8, 8192, 64),                                   # one row of tiles: runs
])
def test_gemm_tiles_in_one_part_for_each_xcd(form, epi, M, N, K):
    test_gemm_forms_and_epilogues(form, epi, M, N, K)


@pytest.mark.parametrize("M,K,n,silu", [
    (512, 1024, 4096, False), (512, 4096, 1024, True), (448, 1024, 1536, False), (447, 1024, 1024, False), (1, 64, 64, False),
    (33, 72, 128, True), (200, 1000, 1536, False), (250, 4104, 1088, True), (320, 4096, 1024, True), (500, 4000, 512, True),
    (640, 1024, 1024, False), (300, 2048, 192, True), (1024, 4096, 1024, True), (2050, 1024, 4096, False),
])
def test_both_gradients_in_one_launch(M, K, n, silu):
    """The bits of the two products, and nothing behind their last rows: tiles of every kind for either, in both orders."""
    lib = seco.load_library()
    P, I = C.c_void_p, C.c_int64
    lib.dec_gemm.argtypes = [C.c_int, C.c_int, P, P, P, P] + [I] * 6 + [P]
    lib.dec_gemm_grads.argtypes = [P] * 6 + [I] * 3 + [P]
    g = torch.Generator(device=DEV).manual_seed(M + K + n)

    def normal(*shape):
        return torch.randn(*shape, generator=g, device=DEV).to(torch.bfloat16)
    dy, w, x, u = normal(M, n), normal(K, n), normal(M, K), normal(M, K)
    dx, dw = normal(M + 1, K), normal(K + 1, n)
    dx2, dw2, s = dx.clone(), dw.clone(), torch.cuda.current_stream().cuda_stream
    ptr = lambda t: t.data_ptr()
    assert lib.dec_gemm(TN, ADD, ptr(x), ptr(dy), ptr(dw), None, K, n, M, K, n, n, s) == 0
    assert lib.dec_gemm(NT, SILU_BWD if silu else STORE, ptr(dy), ptr(w), ptr(dx), ptr(u) if silu else None, M, K, n, n, n, K, s) == 0
    assert lib.dec_gemm_grads(ptr(dy), ptr(w), ptr(dx2), ptr(u) if silu else None, ptr(x), ptr(dw2), M, K, n, s) == 0
    torch.cuda.synchronize()
    assert torch.equal(dx, dx2) and torch.equal(dw, dw2)


@pytest.mark.parametrize("M,K,n,silu", [
    (512, 4096, 1024, True), (512, 1024, 4096, False), (447, 1024, 1024, False), (1, 64, 64, False), (33, 72, 128, True),
    (320, 4096, 1024, True), (1024, 4096, 1024, True), (2050, 1024, 4096, False),
])
def test_first_gradients_in_one_launch(M, K, n, silu):
    """As above where there is nothing to add to yet: what the weight gradient holds before does not matter."""
    lib = seco.load_library()
    P, I = C.c_void_p, C.c_int64
    lib.dec_gemm.argtypes = [C.c_int, C.c_int, P, P, P, P] + [I] * 6 + [P]
    lib.dec_gemm_first_grads.argtypes = [P] * 6 + [I] * 3 + [P]
    g = torch.Generator(device=DEV).manual_seed(M + K + n)
    dy, w, x, u = (torch.randn(*s, generator=g, device=DEV).to(torch.bfloat16) for s in ((M, n), (K, n), (M, K), (M, K)))
    dx, dw = (torch.full(s, float("nan"), device=DEV, dtype=torch.bfloat16) for s in ((M, K), (K, n)))
    dx2, dw2, s = dx.clone(), dw.clone(), torch.cuda.current_stream().cuda_stream
    ptr = lambda t: t.data_ptr()
    assert lib.dec_gemm(TN, STORE, ptr(x), ptr(dy), ptr(dw), None, K, n, M, K, n, n, s) == 0
    assert lib.dec_gemm(NT, SILU_BWD if silu else STORE, ptr(dy), ptr(w), ptr(dx), ptr(u) if silu else None, M, K, n, n, n, K, s) == 0
    assert lib.dec_gemm_first_grads(ptr(dy), ptr(w), ptr(dx2), ptr(u) if silu else None, ptr(x), ptr(dw2), M, K, n, s) == 0
    torch.cuda.synchronize()
    assert torch.equal(dx, dx2) and torch.equal(dw, dw2)


def test_silu_and_its_derivative_at_every_u():
    """Both at all values of u, those whose e^-u leaves fp32 among their neighbours: u out of a product with the identity, one as
    the gradient behind the SiLU.  Error: half an ulp of bf16, 2^-8 of the value at most, and that of e^-u, whose argument is
    rounded to 2^-24 of up to 128: less than 2^-14.  Near u = -1.28 the derivative is a difference of numbers around one (2^-22);
    where e^-u > 2^128 ends fp32 the result is zero instead of |u| 2^-128 at most, |u| < 90 while that counts: 2^-121."""
    lib = seco.load_library()
    P, I = C.c_void_p, C.c_int64
    lib.dec_gemm.argtypes = [C.c_int, C.c_int, P, P, P, P] + [I] * 6 + [P]
    u = torch.arange(65536, device=DEV, dtype=torch.int32).to(torch.int16).view(torch.bfloat16)
    finite = torch.where(torch.isfinite(u), u, torch.zeros_like(u)).view(64, 1024)
    eye, ones = torch.eye(64, device=DEV, dtype=torch.bfloat16), torch.ones(1024, 64, device=DEV, dtype=torch.bfloat16)
    c, act, grad = (torch.empty(64, 1024, device=DEV, dtype=torch.bfloat16) for _ in range(3))
    s = torch.cuda.current_stream().cuda_stream

    def close(x, ref, ud):
        bound = ref.abs() * (2.0 ** -8 + 2.0 ** -14) + torch.where(ud.abs() < 2, 2.0 ** -22, 2.0 ** -121)
        return bool(((x.double() - ref).abs() <= bound).all())
    assert lib.dec_gemm(NN, SILU, eye.data_ptr(), finite.data_ptr(), c.data_ptr(), act.data_ptr(), 64, 1024, 64, 64, 1024, 1024, s) == 0
    ud = finite.double()
    sig = torch.sigmoid(ud)
    assert torch.equal(c, finite) and close(act, ud * sig, ud)
    u = u.view(64, 1024).contiguous()
    assert lib.dec_gemm(NT, SILU_BWD, eye.data_ptr(), ones.data_ptr(), grad.data_ptr(), u.data_ptr(), 64, 1024, 64, 64, 64, 1024, s) == 0
    fin = torch.isfinite(u)
    assert close(grad[fin], (sig * (1 + ud * (1 - sig)))[fin], ud[fin]) and bool(torch.isnan(grad[torch.isnan(u)]).all())


def test_gemm_refuses_what_it_cannot_do():
    lib = seco.load_library()
    I = C.c_int64
    lib.dec_gemm_supported.argtypes = [C.c_int] + [I] * 6
    ok = lib.dec_gemm_supported
    assert ok(NN, 5, 64, 64, 64, 64, 64) and ok(TN, 64, 64, 5, 64, 64, 64)
    assert not ok(NN, 5, 29, 64, 64, 29, 29) and not ok(NN, 5, 64, 96, 96, 64, 64) and not ok(TN, 60, 64, 64, 60, 64, 64)


@pytest.mark.parametrize("first", [False, True])
@pytest.mark.parametrize("M,K,n,silu", [
    (384, 1024, 64, False), (383, 1024, 1536, True), (449, 1024, 512, False), (1001, 512, 576, True), (1472, 256, 2304, False),
    (200, 1536, 1024, False), (8, 6144, 64, False), (775, 640, 1024, False),
    (140, 2560, 192, True), (512, 1024, 2048, False),      # a round of an XCD saved: last tiles of 12 rows, and beside 128 x 128 ones
])
def test_gradients_in_one_launch_with_taller_tiles(M, K, n, silu, first):
    """Around the line where the data gradient takes 64 rows to a tile (96 tiles, rows that fill them or not, weight gradients that do
    or do not fit beside): the bits of the product by itself, and nothing behind its last row."""
    lib = seco.load_library()
    P, I = C.c_void_p, C.c_int64
    entry = lib.dec_gemm_first_grads if first else lib.dec_gemm_grads
    lib.dec_gemm.argtypes = [C.c_int, C.c_int, P, P, P, P] + [I] * 6 + [P]
    entry.argtypes = [P] * 6 + [I] * 3 + [P]
    g = torch.Generator(device=DEV).manual_seed(M + K + n)
    dy, w, x, u, dx, dw = (torch.randn(*s, generator=g, device=DEV).to(torch.bfloat16)
                           for s in ((M, n), (K, n), (M, K), (M, K), (M + 1, K), (K + 1, n)))
    dx2, dw2, s = dx.clone(), dw.clone(), torch.cuda.current_stream().cuda_stream
    ptr = lambda t: t.data_ptr()
    assert lib.dec_gemm(TN, STORE if first else ADD, ptr(x), ptr(dy), ptr(dw), None, K, n, M, K, n, n, s) == 0
    assert lib.dec_gemm(NT, SILU_BWD if silu else STORE, ptr(dy), ptr(w), ptr(dx), ptr(u) if silu else None, M, K, n, n, n, K, s) == 0
    assert entry(ptr(dy), ptr(w), ptr(dx2), ptr(u) if silu else None, ptr(x), ptr(dw2), M, K, n, s) == 0
    torch.cuda.synchronize()
    assert torch.equal(dx, dx2) and torch.equal(dw, dw2)
