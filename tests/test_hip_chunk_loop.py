"""GPU parity of the end-to-end SeCO / SpaCO step (Alg. 1, Alg. 2 over a multi-layer decoder) against the
fp64 model oracle: same seeded parameters and tokens on both sides, parameter gradients compared tensor by
tensor as max|x - ref| / max|ref|.

Tolerances: fp32 run 5e-4 (the kernels' own bar is 1e-4 per call; here three layers of fp32 GEMMs, norms and
the relay stack on top of each other), bf16 run 6e-2 (every activation and every relayed gradient is rounded to
bf16, 2^-9 relative each, through about 20 roundings per chain)."""
import pytest
import torch

from oracle import model as om

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


def _setup(cfg, seed, B, N, dtype):
    from paper_2505_16710_amd.chunk_loop import ChunkedDecoder
    p64 = om.init_params(cfg, seed)
    if dtype is torch.bfloat16:        # both sides start from the same bf16-representable parameters
        p64 = {n: t.detach().to(torch.bfloat16).to(torch.float64).requires_grad_() for n, t in p64.items()}
    pg = {n: t.detach().to(dtype).to(DEV).requires_grad_() for n, t in p64.items()}
    g = torch.Generator().manual_seed(seed + 100)
    tok = torch.randint(0, cfg.vocab, (B, N), generator=g)
    tgt = torch.randint(0, cfg.vocab, (B, N), generator=g)
    dec = ChunkedDecoder(pg, cfg.n_layers, cfg.n_q_heads, cfg.n_kv_heads, cfg.head_dim,
                         rope_base=cfg.rope_base if cfg.rope_base > 1.0 else None)
    return p64, dec, tok, tgt


def _compare(g_ref, g_gpu, tol):
    worst = 0.0
    for n, ref in g_ref.items():
        x = g_gpu[n].detach().to(torch.float64).cpu()
        err = float((x - ref).abs().max() / ref.abs().max().clamp_min(1e-30))
        worst = max(worst, err)
        assert err < tol, (n, err)
    return worst


F32_CFG = om.ModelConfig(n_layers=3, d_model=64, n_q_heads=4, n_kv_heads=2, head_dim=32, d_ff=96, vocab=29)
BF16_CFG = om.ModelConfig(n_layers=2, d_model=64, n_q_heads=2, n_kv_heads=1, head_dim=128, d_ff=96, vocab=29)


@pytest.mark.parametrize("N,C", [(96, 24), (100, 32)])
def test_seco_step_fp32_matches_whole_sequence_gradient(N, C):
    p64, dec, tok, tgt = _setup(F32_CFG, 5, 2, N, torch.float32)
    loss_ref, g_ref = om.monolithic_grads(F32_CFG, p64, tok, tgt)
    loss, g = dec.step(tok.to(DEV), tgt.to(DEV), C)
    assert abs(loss - float(loss_ref)) < 1e-4 * abs(float(loss_ref))
    _compare(g_ref, g, 5e-4)


def test_spaco_step_fp32_matches_oracle():
    N, C, sel, f = 160, 32, [4, 2, 1], 5.0 / 3.0
    p64, dec, tok, tgt = _setup(F32_CFG, 7, 2, N, torch.float32)
    _, g_ref = om.spaco_grads(F32_CFG, p64, tok, tgt, C, sel, f)
    _, g = dec.step(tok.to(DEV), tgt.to(DEV), C, selected=sel, factor=f)
    _compare(g_ref, g, 5e-4)
    # the compound factor really is exercised: with factor 1 the reference differs visibly
    _, g_one = om.spaco_grads(F32_CFG, p64, tok, tgt, C, sel, 1.0)
    assert max(float((g_one[n] - g_ref[n]).abs().max() / g_ref[n].abs().max()) for n in g_ref) > 1e-2


def test_seco_step_bf16_matmul_kernels():
    N, C = 256, 64
    p64, dec, tok, tgt = _setup(BF16_CFG, 9, 1, N, torch.bfloat16)
    _, g_ref = om.monolithic_grads(BF16_CFG, p64, tok, tgt)
    _, g = dec.step(tok.to(DEV), tgt.to(DEV), C)
    _compare(g_ref, g, 6e-2)


def test_spaco_step_bf16_matmul_kernels():
    N, C, sel, f = 320, 64, [4, 3, 0], 5.0 / 3.0
    p64, dec, tok, tgt = _setup(BF16_CFG, 11, 1, N, torch.bfloat16)
    _, g_ref = om.spaco_grads(BF16_CFG, p64, tok, tgt, C, sel, f)
    _, g = dec.step(tok.to(DEV), tgt.to(DEV), C, selected=sel, factor=f)
    _compare(g_ref, g, 6e-2)


@pytest.mark.parametrize("dtype,cfg", [(torch.float32, F32_CFG), (torch.bfloat16, BF16_CFG)])
def test_keeping_attention_outputs_gives_identical_gradients(dtype, cfg):
    """Stage 2 may take O and LSE from stage 1 instead of running the attention forward again: same values
    (deterministic kernels, same inputs), hence bit-identical gradients, for SeCO and SpaCO."""
    p64, dec, tok, tgt = _setup(cfg, 13, 1, 256, dtype)
    tok, tgt = tok.to(DEV), tgt.to(DEV)
    for kw in ({}, {"selected": [3, 1, 0], "factor": 4 / 3}):
        _, g_a = dec.step(tok, tgt, 64, **kw)
        g_a = {n: t.clone() for n, t in g_a.items()}
        _, g_b = dec.step(tok, tgt, 64, keep_attention_outputs=True, **kw)
        for n in g_a:
            assert torch.equal(g_a[n], g_b[n]), n


@pytest.mark.parametrize("dtype,cfg,N", [(torch.float32, F32_CFG, 200), (torch.bfloat16, BF16_CFG, 256)])
@pytest.mark.parametrize("kw", [{}, {"keep_attention_outputs": True}])
def test_losses_of_a_step_that_visits_every_chunk(dtype, cfg, N, kw):
    """They come from stage 2; with a chunk left out, from stage 1: the same bits (same launches on the same inputs)."""
    _, dec, tok, tgt = _setup(cfg, 17, 1, N, dtype)
    tok, tgt = tok.to(DEV), tgt.to(DEV)
    every, _ = dec.step(tok, tgt, 64, **kw)
    picked, _ = dec.step(tok, tgt, 64, selected=[0, 1, 2, 3], factor=1.0, **kw)
    some, _ = dec.step(tok, tgt, 64, selected=[3, 1, 0], factor=4 / 3, **kw)
    assert every == picked == some


@pytest.mark.parametrize("B", [1, 2])
def test_tokens_and_targets_of_any_stride(B):
    _, dec, tok, tgt = _setup(F32_CFG, 20, B, 96, torch.float32)
    loss, g = dec.step(tok.to(DEV), tgt.to(DEV), 40)
    g = {n: t.clone() for n, t in g.items()}
    strided = [torch.stack((t, t * 0 + 1), -1).to(DEV).flatten(1)[:, ::2] for t in (tok, tgt)]
    assert strided[0].stride(1) == 2
    loss_s, g_s = dec.step(*strided, 40)
    assert loss_s == loss
    for n in g:
        assert torch.equal(g_s[n], g[n]), n


@pytest.mark.parametrize("keep", [False, True])
def test_step_that_leaves_the_last_chunk_out(keep):
    """Stage 2 then does not start with the last chunk, and stage 1 has to run it: the same losses, and the oracle's gradients.  With
    the last chunk as the only one stage 1 runs the others for their cache rows."""
    _, dec, tok, tgt = _setup(F32_CFG, 19, 1, 120, torch.float32)
    p64, tok_g, tgt_g = {n: t.detach().double().cpu().requires_grad_() for n, t in dec.p.items()}, tok.to(DEV), tgt.to(DEV)
    every, _ = dec.step(tok_g, tgt_g, 32, keep_attention_outputs=keep)
    for sel in ([2, 0], [3], [0]):
        loss, g = dec.step(tok_g, tgt_g, 32, selected=sel, factor=1.5, keep_attention_outputs=keep)
        assert loss == every, sel
        _, g_ref = om.spaco_grads(F32_CFG, p64, tok, tgt, 32, sel, 1.5)
        _compare(g_ref, g, 5e-4)


@pytest.mark.parametrize("dtype,cfg,tol,transposed,keep", [
    (torch.float32, F32_CFG, 5e-4, False, False), (torch.float32, F32_CFG, 5e-4, False, True),
    (torch.bfloat16, BF16_CFG, 6e-2, False, False), (torch.bfloat16, BF16_CFG, 6e-2, False, True),
    (torch.bfloat16, BF16_CFG, 6e-2, True, False)])
def test_alg1_walks_the_chunks_it_is_given(dtype, cfg, tol, transposed, keep):
    """The relay over four chunks, the last one ragged.  chunk_len is the caller's bound on the activations alive: a step takes no
    more memory, and gives the same bits, than one whose stage1_chunk_len repeats it, and less than the sequence as one chunk."""
    N, C = 230, 64
    p64, dec, tok, tgt = _setup(cfg, 36, 2, N, dtype)
    loss_ref, g_ref = om.monolithic_grads(cfg, p64, tok, tgt)
    tok, tgt = tok.to(DEV), tgt.to(DEV)

    def step(c, c1):
        for _ in range(2):                      # (the first one brings what outlives a step)
            torch.cuda.reset_peak_memory_stats()
            before = torch.cuda.memory_allocated()
            loss, g = dec.step(tok, tgt, c, stage1_chunk_len=c1, keep_attention_outputs=keep, transposed_backward=transposed)
            peak = torch.cuda.max_memory_allocated() - before
            g = {n: t.double().cpu() for n, t in g.items()}
            for t in dec.p.values():
                t.grad = None
        return loss, g, peak
    loss, g, peak = step(C, None)
    assert abs(loss - float(loss_ref)) < (1e-4 if dtype is torch.float32 else 2e-2) * abs(float(loss_ref))
    _compare(g_ref, g, tol)
    again, g_again, peak_again = step(C, C)
    assert loss == again and peak == peak_again
    for n in g:
        assert torch.equal(g[n], g_again[n]), n
    assert peak < step(N, None)[2]


@pytest.mark.parametrize("transposed,wide_tail", [(True, False), (False, True), (True, True)])
def test_losses_of_stage_2_in_the_transposed_order_and_behind_a_wide_tail(transposed, wide_tail):
    """The same, with the transposed backward order and with an fp32 final norm and head behind the bf16 body; a ragged last chunk."""
    _, dec, tok, tgt = _setup(BF16_CFG, 18, 2, 250, torch.bfloat16)
    for n in ("norm_f", "head") if wide_tail else ():
        dec.p[n] = om.init_params(BF16_CFG, 34)[n].detach().to(torch.float32).to(DEV).requires_grad_()
    tok, tgt = tok.to(DEV), tgt.to(DEV)
    every, _ = dec.step(tok, tgt, 64, transposed_backward=transposed)
    picked, _ = dec.step(tok, tgt, 64, selected=[0, 1, 2, 3], factor=1.0, transposed_backward=transposed)
    some, _ = dec.step(tok, tgt, 64, selected=[3, 1, 0], factor=4 / 3, transposed_backward=transposed)
    assert every == picked == some


def test_whole_sequence_stage1_with_kept_outputs_matches_oracle():
    """Stage 1 as one plain forward over the whole sequence, stage 2 from its kept O / LSE: same gradients as the
    oracle's Alg. 1 / Alg. 2 (to the usual tolerance; the launches differ in shape from the chunked stage 1)."""
    N, C = 192, 32
    p64, dec, tok, tgt = _setup(F32_CFG, 15, 2, N, torch.float32)
    _, g_ref = om.monolithic_grads(F32_CFG, p64, tok, tgt)
    _, g = dec.step(tok.to(DEV), tgt.to(DEV), C, keep_attention_outputs=True, stage1_chunk_len=N)
    _compare(g_ref, g, 5e-4)
    sel, f = [5, 3, 0], 2.0
    _, g_ref = om.spaco_grads(F32_CFG, p64, tok, tgt, C, sel, f)
    _, g = dec.step(tok.to(DEV), tgt.to(DEV), C, selected=sel, factor=f, keep_attention_outputs=True, stage1_chunk_len=N)
    _compare(g_ref, g, 5e-4)
    # bf16 matrix-core kernels
    p64, dec, tok, tgt = _setup(BF16_CFG, 16, 1, 256, torch.bfloat16)
    _, g_ref = om.monolithic_grads(BF16_CFG, p64, tok, tgt)
    _, g = dec.step(tok.to(DEV), tgt.to(DEV), 64, keep_attention_outputs=True, stage1_chunk_len=256)
    _compare(g_ref, g, 6e-2)


@pytest.mark.parametrize("dtype,cfg,tol", [(torch.float32, F32_CFG, 5e-4), (torch.bfloat16, BF16_CFG, 6e-2)])
def test_column_weighted_dq_step_matches_oracle(dtype, cfg, tol):
    """Alg. 2 with, beyond the paper, a dQ that visits only some chunks, a different weight vector in every layer
    of every call (fixed here; a training loop would draw them)."""
    N, C, sel, f = 320, 64, [4, 3, 1, 0], 1.25
    p64, dec, tok, tgt = _setup(cfg, 13, 1, N, dtype)

    def wq(j, l):
        g = torch.Generator().manual_seed(1000 * j + l)
        w = [float(x) * 2.0 for x in (torch.rand(j, generator=g) < 0.5)] + [1.0]
        return w
    _, g_ref = om.spaco_grads(cfg, p64, tok, tgt, C, sel, f, dq_weights=wq)
    _, g = dec.step(tok.to(DEV), tgt.to(DEV), C, selected=sel, factor=f, dq_weights=wq)
    _compare(g_ref, g, tol)
    _, g_dense = om.spaco_grads(cfg, p64, tok, tgt, C, sel, f)
    assert max(float((g_dense[n] - g_ref[n]).abs().max() / g_ref[n].abs().max()) for n in g_ref) > 1e-2


@pytest.mark.parametrize("dtype,base_cfg,tol", [(torch.float32, F32_CFG, 5e-4), (torch.bfloat16, BF16_CFG, 6e-2)])
def test_step_with_rotary_embedding_matches_oracle(dtype, base_cfg, tol):
    """Queries rotated by rope_rotate, keys rotated on their way into the cache (kv_append_rope), the key gradient
    turned back at the read-out (kvgrad_readout_rope): SeCO against whole-sequence training, SpaCO against Alg. 2."""
    import dataclasses
    cfg = dataclasses.replace(base_cfg, rope_base=10000.0)
    N, C = 320, 64
    p64, dec, tok, tgt = _setup(cfg, 15, 1, N, dtype)
    _, g_ref = om.monolithic_grads(cfg, p64, tok, tgt)
    _, g = dec.step(tok.to(DEV), tgt.to(DEV), C, keep_attention_outputs=True)
    _compare(g_ref, g, tol)
    _, g_plain = om.monolithic_grads(base_cfg, p64, tok, tgt)          # the embedding is really there
    assert max(float((g_plain[n] - g_ref[n]).abs().max() / g_ref[n].abs().max()) for n in g_ref) > 1e-2
    sel, f = [4, 2, 1], 5.0 / 3.0
    _, g_ref = om.spaco_grads(cfg, p64, tok, tgt, C, sel, f)
    _, g = dec.step(tok.to(DEV), tgt.to(DEV), C, selected=sel, factor=f)
    _compare(g_ref, g, tol)


def test_seco_step_with_the_transposed_backward_order_matches_whole_sequence_training():
    """Alg. 1 with every layer's attention backward in the transposed order (seco_chunk_attn_bwd_gather): parameter
    gradients against ordinary whole-sequence training, ragged last chunk included, and against the accumulating
    order to rounding."""
    cfg, tol = BF16_CFG, 6e-2
    N, C = 448, 128
    p64, dec, tok, tgt = _setup(cfg, 19, 2, N, torch.bfloat16)
    _, g_ref = om.monolithic_grads(cfg, p64, tok, tgt)
    loss_t, g_t = dec.step(tok.to(DEV), tgt.to(DEV), C, transposed_backward=True)
    _compare(g_ref, g_t, tol)
    loss_a, g_a = dec.step(tok.to(DEV), tgt.to(DEV), C)
    assert loss_t == loss_a
    for n in g_a:
        d = (g_t[n].float() - g_a[n].float()).abs().max() / g_a[n].float().abs().max()
        assert float(d) < 2e-2, (n, float(d))


def test_spaco_step_with_the_transposed_backward_order_matches_oracle():
    """Alg. 2 with every layer's attention backward in the transposed order (row weights 1 / factor / 0)."""
    cfg, tol = BF16_CFG, 6e-2
    N, C = 320, 64
    p64, dec, tok, tgt = _setup(cfg, 23, 1, N, torch.bfloat16)
    sel, f = [4, 2, 1], 5.0 / 3.0
    _, g_ref = om.spaco_grads(cfg, p64, tok, tgt, C, sel, f)
    _, g = dec.step(tok.to(DEV), tgt.to(DEV), C, selected=sel, factor=f, transposed_backward=True)
    _compare(g_ref, g, tol)


@pytest.mark.parametrize("widths", [(96, 160, 64), (160, 64, 96)])
def test_step_with_mlp_widths_that_differ_between_layers(widths):
    p64, dec, tok, tgt = _setup(F32_CFG, 29, 1, 64, torch.float32)
    g = torch.Generator().manual_seed(30)
    for l, ff in enumerate(widths):
        for n, shape in ((f"l{l}.w1", (F32_CFG.d_model, ff)), (f"l{l}.w2", (ff, F32_CFG.d_model))):
            p64[n] = (torch.randn(shape, generator=g, dtype=torch.float64) * shape[0] ** -0.5).requires_grad_()
            dec.p[n] = p64[n].detach().to(torch.float32).to(DEV).requires_grad_()
    _, g_ref = om.monolithic_grads(F32_CFG, p64, tok, tgt)
    _, g = dec.step(tok.to(DEV), tgt.to(DEV), 24)
    _compare(g_ref, g, 5e-4)


def test_step_with_gains_of_one_element_or_a_narrower_type():
    """A gain multiplies its rows by broadcasting: one element, leading ones and (in fp32) bf16 values are gains too."""
    p64, dec, tok, tgt = _setup(F32_CFG, 31, 1, 64, torch.float32)
    gains = {"l0.norm1": torch.tensor([0.75]), "l1.norm2": torch.tensor(1.25), "norm_f": torch.tensor([[[1.5]]]),
             "l2.norm1": (1 + torch.arange(64) / 64).to(torch.bfloat16), "l0.norm2": (1 + torch.arange(64) / 64)[None, None]}
    for n, t in gains.items():
        p64[n] = t.to(torch.float64).requires_grad_()
        dec.p[n] = t.to(DEV).requires_grad_()
    _, g_ref = om.monolithic_grads(F32_CFG, p64, tok, tgt)
    _, g = dec.step(tok.to(DEV), tgt.to(DEV), 24)
    for n, t in gains.items():
        assert g[n].shape == t.shape and g[n].dtype == t.dtype
    _compare({n: t for n, t in g_ref.items() if n != "l2.norm1"}, g, 5e-4)
    _compare({"l2.norm1": g_ref["l2.norm1"]}, g, 5e-4 + 2.0 ** -8)     # rounded to bf16 once more


def test_step_with_an_fp32_final_norm_and_head_behind_a_bf16_body():
    p64, dec, tok, tgt = _setup(BF16_CFG, 33, 2, 192, torch.bfloat16)
    for n in ("norm_f", "head"):
        p64[n] = om.init_params(BF16_CFG, 34)[n].detach().to(torch.float32).to(torch.float64).requires_grad_()
        dec.p[n] = p64[n].detach().to(torch.float32).to(DEV).requires_grad_()
    loss_ref, g_ref = om.monolithic_grads(BF16_CFG, p64, tok, tgt)
    loss, g = dec.step(tok.to(DEV), tgt.to(DEV), 64)
    assert g["head"].dtype == g["norm_f"].dtype == torch.float32
    assert abs(loss - float(loss_ref)) < 1e-2 * abs(float(loss_ref))
    _compare(g_ref, g, 6e-2)


@pytest.mark.parametrize("dtype,cfg", [(torch.float32, F32_CFG), (torch.bfloat16, BF16_CFG)])
def test_step_with_parameters_at_any_address(dtype, cfg):
    """Parameters that are pieces of one buffer start on no 16-byte boundary; the gradients do not change."""
    _, dec, tok, tgt = _setup(cfg, 35, 1, 128, dtype)
    _, g_ref = dec.step(tok.to(DEV), tgt.to(DEV), 64)
    flat = torch.zeros(1 + sum(t.numel() + -t.numel() % 8 for t in dec.p.values()), dtype=dtype, device=DEV)
    at = 1
    for n, t in list(dec.p.items()):
        piece = flat[at:at + t.numel()].view(t.shape)
        piece.copy_(t.detach())
        dec.p[n] = piece.requires_grad_()
        assert piece.data_ptr() % 16 != 0
        at += t.numel() + -t.numel() % 8
    _, g = dec.step(tok.to(DEV), tgt.to(DEV), 64)
    for n in g_ref:
        assert torch.equal(g[n], g_ref[n]), n


@pytest.mark.parametrize("transposed", [False, True])
@pytest.mark.parametrize("rope", [False, True])
def test_chunk_attention_composes_with_autograd(rope, transposed):
    """LayerState, Rope and ChunkAttention between framework operators: Alg. 1 over one layer (projections, attention, a
    loss of the outputs) leaves the gradients of whole-sequence attention at the weights and at the inputs."""
    from paper_2505_16710_amd.chunk_loop import ChunkAttention, LayerState, Rope
    B_, N, C, Hq, Hkv, D, dm, base = 1, 160, 64, 2, 1, 128, 64, 10000.0
    scale = D ** -0.5
    gen = torch.Generator().manual_seed(41)
    rnd = lambda *s: torch.randn(*s, generator=gen, dtype=torch.float64).to(torch.bfloat16).double()
    x, t = rnd(B_, N, dm), rnd(B_, N, Hq * D)
    w = {n: rnd(dm, h * D) * dm ** -0.5 for n, h in (("q", Hq), ("k", Hkv), ("v", Hkv))}
    w = {n: v.to(torch.bfloat16).double() for n, v in w.items()}

    def heads(y, h):
        return y.view(B_, -1, h, D).transpose(1, 2)
    ref = {n: v.clone().requires_grad_() for n, v in {**w, "x": x}.items()}
    q, k, v = (heads(ref["x"] @ ref[n], h) for n, h in (("q", Hq), ("k", Hkv), ("v", Hkv)))
    if rope:
        q, k = om._rope(q, 0, base), om._rope(k, 0, base)
    (om._attend(q, k, v, 0, scale).transpose(1, 2).reshape(B_, N, -1) * t).sum().backward()

    gpu = {n: v.to(torch.bfloat16).to(DEV).requires_grad_() for n, v in {**w, "x": x}.items()}
    tg, hooked = t.to(torch.bfloat16).to(DEV), []
    gpu["q"].register_hook(lambda g: hooked.append(g.shape))
    st = LayerState(B_, Hkv, N, D, torch.bfloat16, DEV)
    if transposed:
        st.enable_gather(B_, Hq, N, D, torch.bfloat16, DEV)

    def chunk(s0):
        xc = gpu["x"][:, s0:s0 + C]
        qc, kc, vc = (heads(xc @ gpu[n], h) for n, h in (("q", Hq), ("k", Hkv), ("v", Hkv)))
        if rope:
            qc = Rope.apply(qc, s0, base)
        o = ChunkAttention.apply(qc, kc, vc, st, s0, scale, None, 0, None, None, base if rope else None)
        return (o.transpose(1, 2).reshape(B_, xc.shape[1], -1) * tg[:, s0:s0 + C]).float().sum()
    from paper_2505_16710_amd import kvgrad_zero
    starts = list(range(0, N, C))
    with torch.no_grad():
        for s0 in starts:
            chunk(s0)
    kvgrad_zero(st.gk, st.gv)
    for s0 in reversed(starts):
        chunk(s0).backward()
    assert len(hooked) == len(starts)
    _compare({n: v.grad for n, v in ref.items()}, {n: v.grad for n, v in gpu.items()}, 6e-2)


def test_step_whose_products_are_partly_the_frameworks():
    """An MLP 8192 wide: the gradient of w2 is taller than the library's own product is used for, the others are not; with
    more rows, forward and backward products cross the line too, and agree with those of shorter chunks to rounding."""
    import dataclasses
    cfg = dataclasses.replace(BF16_CFG, n_layers=1, d_model=512, d_ff=8192, vocab=64)
    p64, dec, tok, tgt = _setup(cfg, 37, 1, 128, torch.bfloat16)
    _, g_ref = om.monolithic_grads(cfg, p64, tok, tgt)
    _, g = dec.step(tok.to(DEV), tgt.to(DEV), 64)
    _compare(g_ref, g, 6e-2)
    gen = torch.Generator().manual_seed(38)
    tok, tgt = (torch.randint(0, cfg.vocab, (1, 4608), generator=gen).to(DEV) for _ in range(2))
    loss_a, g_a = dec.step(tok, tgt, 4608)      # 4608 x 512 x 8192 multiply-adds
    loss_b, g_b = dec.step(tok, tgt, 512)
    assert abs(loss_a - loss_b) < 1e-3 * loss_b
    for n in g_a:
        assert float((g_a[n].float() - g_b[n].float()).norm() / g_b[n].float().norm()) < 2e-2, n


@pytest.mark.parametrize("dtype,cfg", [(torch.float32, F32_CFG), (torch.bfloat16, BF16_CFG)])
@pytest.mark.parametrize("at,token", [(0, 29), (100, -30), (127, 1 << 40)])
def test_tokens_outside_the_embedding_table_are_refused(dtype, cfg, at, token):
    """In any chunk and schedule, also where no loss could tell (targets left out from that position on); negative ones within the
    table count from its end, and a step behind a refused one is what it was."""
    _, dec, tok, tgt = _setup(cfg, 23, 1, 128, dtype)
    tok, tgt = tok.to(DEV), tgt.to(DEV)
    loss, g = dec.step(tok, tgt, 32)
    g = {n: t.clone() for n, t in g.items()}
    bad, some = tok.clone(), tgt.clone()
    bad[0, at], some[0, at:] = token, -100
    for kw in ({}, {"selected": [2, 0], "factor": 2.0}, {"selected": [3]}, {"keep_attention_outputs": True}, {"stage1_chunk_len": 128}):
        for targets in (tgt, some):
            with pytest.raises(IndexError):
                dec.step(bad, targets, 32, **kw)
            assert all(t.grad is None for t in dec.p.values())
    again, g_again = dec.step(torch.where(tok % 2 == 0, tok - cfg.vocab, tok), tgt, 32)
    assert again == loss and all(torch.equal(g[n], g_again[n]) for n in g)
