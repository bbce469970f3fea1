"""SeCO / SpaCO training step of a small decoder, driven through the C ABI (Alg. 1 and Alg. 2 end to end).

The attention of every layer, its backward and the whole KV-gradient relay run in the HIP library:
each layer owns a KV cache and a pair of fp32 KV-gradient buffers that live for the whole step, the
forward of a chunk is `seco_chunk_attn_fwd` against the cache, its backward is `seco_chunk_attn_bwd` /
`spaco_chunk_attn_bwd`, which deposits the chunk's dK/dV on every visible cache row, and the gradient
handed to the chunk's own recomputed K/V is simply the chunk's rows of those buffers (they hold what
the later chunks deposited plus the chunk's own diagonal block: the relay of Alg. 1, `m_i.grad <-
m'_i.grad`), read out by `kvgrad_readout`; new keys / values enter the cache through `kv_append`.  Under SpaCO the deposits on earlier selected chunks carry the compensation
factor, so a chain through p caches is scaled by factor^p (Sec. 5).

The projections and the MLP, the residual adds, norms, SiLU, loss and embedding gradient around the attention are
kernels of the library too (gemm_bf16.hip, decoder.hip), the derivatives are written out instead of being recorded, and
a chunk is launched by one call of the binding's extension module (chunk_step_ext.cpp): at the row counts of a chunk a
step is bound by the number of launches and the host time behind each (with autograd and framework operators, 27 ms for
two layers over 4096 tokens in chunks of 512, of which the GPU worked 14).  Products whose type or alignment the
library's kernel does not take (fp32, row lengths that are not multiples of 8) go through the framework's.  Only one
chunk's activations are alive at a time, as in the paper.  There is no CPU path.

Model (fixed here so that a checker can build the same function): pre-norm decoder, RMSNorm with
eps 1e-6, grouped-query causal attention (optionally with rotary position embedding), MLP x + silu(h W1) W2, final
RMSNorm, linear head, cross-entropy summed over tokens.  Parameter names: emb, head, norm_f and
l{i}.norm1, l{i}.norm2, l{i}.wq, l{i}.wk, l{i}.wv, l{i}.wo, l{i}.w1, l{i}.w2, all stored [in, out].
"""
from __future__ import annotations

import torch

from . import binding as _b


class ChunkedDecoder:
    """Holds the parameters (dict name -> leaf tensor on the GPU) and runs SeCO / SpaCO steps."""

    def __init__(self, params, n_layers, n_q_heads, n_kv_heads, head_dim, rope_base=None):
        self.p = params
        self.rope_base = rope_base      # rotary embedding of queries and keys (keys are cached rotated), or None
        self.n_layers, self.Hq, self.Hkv, self.D = n_layers, n_q_heads, n_kv_heads, head_dim
        self.scale = float(head_dim) ** -0.5
        _b.load_library()          # fail here, loudly, if the HIP library has not been built

    def step(self, tokens, targets, chunk_len, selected=None, factor=1.0, keep_attention_outputs=False,
             stage1_chunk_len=None, dq_weights=None, transposed_backward=False):
        """One SeCO step (selected is None: Alg. 1) or SpaCO step (Alg. 2, `selected` chunk indices,
        relay factor `factor`).  Returns (sum of the chunk losses from stage 1, {name: gradient}).

        keep_attention_outputs: stage 1 keeps every layer's O and LSE (2 + 4/D bytes per query element: with 288 GB
        of HBM that is cheap), and the rebuilt chunks of stage 2 take them back instead of running the attention
        forward again; the gradients are bit-identical to the recomputing schedule.
        stage1_chunk_len: chunk length of the inference pass only (default chunk_len).  Stage 1 holds no graph, so on a
        GPU with room for one layer's activations of the whole sequence it can run as a single chunk (a plain
        prefill); together with keep_attention_outputs, stage 2 then launches backward kernels only.  The caches
        and kept outputs are then produced by differently shaped launches, so gradients agree with the chunked
        stage 1 to rounding, not bit for bit.
        dq_weights: optional callable (chunk j, layer l) -> one non-negative weight per chunk 0..j (or None): the dQ
        of that attention call visits only the chunks with a non-zero weight and scales their terms
        (spaco_chunk_attn_bwd_sparse_dq; not part of the paper).  For unbiased gradients the weights must have
        expectation 1 and be drawn independently for every layer of a call.
        transposed_backward: the attention backward in the transposed order (seco_chunk_attn_bwd_gather, under Alg. 2
        spaco_chunk_attn_bwd_gather; bf16 parameters): same gradients up to the order of summation."""
        p = self.p
        B, N = tokens.shape
        dtype, dev = p["emb"].dtype, p["emb"].device
        for t in (tokens, targets):
            if t.dim() != 2 or t.shape[0] != B or t.shape[1] < N:
                raise ValueError("tokens and targets must be [batch, tokens], one target per token")
            if t.dtype.is_floating_point or t.dtype.is_complex or t.dtype == torch.bool:
                raise TypeError("tokens and targets must be integers")
            if t.device != dev:
                raise ValueError("tokens and targets must be on the parameters' device")
        starts = list(range(0, N, chunk_len))
        if transposed_backward:
            if dq_weights is not None or dtype != torch.bfloat16:
                raise ValueError("the transposed backward order takes bf16 parameters and the exact dQ")
            if selected is not None and chunk_len % 64 != 0:
                raise ValueError("Alg. 2 in the transposed order needs a chunk length that is a multiple of 64")
        for t in p.values():
            t.grad = None
        c1 = stage1_chunk_len or chunk_len
        picked = None if selected is None else {int(i) for i in selected}
        order = range(len(starts) - 1, -1, -1) if selected is None else sorted(picked, reverse=True)
        if keep_attention_outputs and any(starts[j] // c1 != (min(starts[j] + chunk_len, N) - 1) // c1 for j in order):
            raise ValueError("kept attention outputs: every chunk must lie within one chunk of stage 1")
        names = ["emb", "head", "norm_f"] + [f"l{l}.{n}" for l in range(self.n_layers)
                                             for n in ("norm1", "norm2", "wq", "wk", "wv", "wo", "w1", "w2")]
        ext = _b._ext or _b._load_ext()
        with torch.no_grad():
            run = ext.step_new((self.n_layers, self.Hq, self.Hkv, self.D, self.scale, self.rope_base, B, N, min(c1, N),
                                min(chunk_len, N), transposed_backward), [p[n] for n in names])
            tokens, targets = tokens.to(torch.int64), targets.to(torch.int64)
            losses = torch.empty(N * B, dtype=torch.float32, device=dev)        # one per token, in stage-1 order
            for s0 in range(0, N, c1):                                      # stage 1: inference over all chunks
                ext.step_infer(run, tokens, targets, s0, min(s0 + c1, N), losses, keep_attention_outputs)
            ext.step_zero(run)
            for j in order:                                                 # stage 2: rebuild + back-propagate
                w = wq = None
                if transposed_backward:     # weights of this and the later row chunks: 1, and the factor on selected ones
                    if selected is not None:
                        w = _b.spaco_gather_row_weights(picked, j, len(starts), float(factor))
                elif selected is not None:
                    w = _b.spaco_chunk_weights(order, j, factor)
                if dq_weights is not None:
                    wq = [dq_weights(j, l) for l in range(self.n_layers)]
                ext.step_train(run, tokens, targets, starts[j], min(starts[j] + chunk_len, N), keep_attention_outputs, w,
                               chunk_len, wq)
            total, grads = float(losses.sum()), dict(zip(names, ext.step_grads(run)))
        # every parameter's gradient, also left in .grad (None there if no chunk reached it)
        out = {}
        for n, t in p.items():
            g = grads.get(n)
            if g is not None and t.requires_grad:
                t.grad = out[n] = g
            else:
                out[n] = torch.zeros_like(t)
        return total, out
