"""SeCO / SpaCO training step of a small decoder, driven through the C ABI (Alg. 1 and Alg. 2 end to end).

The attention of every layer, its backward and the whole KV-gradient relay run in the HIP library:
each layer owns a KV cache and a pair of fp32 KV-gradient buffers that live for the whole step, the
forward of a chunk is `seco_chunk_attn_fwd` against the cache, its backward is `seco_chunk_attn_bwd` /
`spaco_chunk_attn_bwd`, which deposits the chunk's dK/dV on every visible cache row, and the gradient
handed to the chunk's own recomputed K/V is simply the chunk's rows of those buffers (they hold what
the later chunks deposited plus the chunk's own diagonal block: the relay of Alg. 1, `m_i.grad <-
m'_i.grad`), read out by `kvgrad_readout`; new keys / values enter the cache through `kv_append`.  Under
SpaCO the deposits on earlier selected chunks carry the compensation factor, so a chain through p caches is
scaled by factor^p (Sec. 5).

The projections and the MLP, the residual adds, norms, SiLU, loss and embedding gradient around the attention are
kernels of the library too (gemm_bf16.hip, decoder.hip), the derivatives are written out instead of being recorded, and
a chunk is launched by one call of the binding's extension module (chunk_step_ext.cpp): at the row counts of a chunk a
step is bound by the number of launches and the host time behind each (with autograd and framework operators, 27 ms for
two layers over 4096 tokens in chunks of 512, of which the GPU worked 14; 3.4 now).  Products whose type or alignment
the library's kernel does not take (fp32, row lengths that are not multiples of 8) and large ones, which the framework's
kernels do faster, go through the framework's.  Only one chunk's activations are alive at a time, as in the paper.
There is no CPU path.  (LayerState, ChunkAttention and Rope are the same attention as autograd functions.)

Parameters are bf16 or fp32 tensors on one GPU, all of one type, with two exceptions: gains may be of a narrower one, and
behind a bf16 body norm_f and head may both be fp32.  Anything else that does not fit is refused before it reaches a
kernel.

Model (fixed here so that a checker can build the same function): pre-norm decoder, RMSNorm with
eps 1e-6, grouped-query causal attention (optionally with rotary position embedding), MLP x + silu(h W1) W2, final
RMSNorm, linear head, cross-entropy summed over tokens.  Parameter names: emb, head, norm_f and
l{i}.norm1, l{i}.norm2, l{i}.wq, l{i}.wk, l{i}.wv, l{i}.wo, l{i}.w1, l{i}.w2, all stored [in, out].
"""
from __future__ import annotations

import torch

from . import binding as _b


# ---- the attention of one layer as an autograd function, for models whose other parts are framework operators ----------
# (ChunkedDecoder drives the same calls natively.)

class LayerState:
    """KV cache (storage dtype) and fp32 KV-gradient buffers of one layer, [B, Hkv, N, D]."""

    def __init__(self, B, Hkv, N, D, dtype, device):
        self.k = torch.zeros(B, Hkv, N, D, dtype=dtype, device=device)
        self.v = torch.zeros_like(self.k)
        self.gk = torch.empty(B, Hkv, N, D, dtype=torch.float32, device=device)
        self.gv = torch.empty_like(self.gk)
        self.kept = {}      # q_start -> (O, LSE) of stage 1, when attention outputs are kept for stage 2
        self.gather = None  # transposed backward order: (Q, dO, O, dQ of the layer, row statistics)
        self.gather_rows = None   # ... under Alg. 2: (selected chunks, factor, chunk length, number of chunks)

    def enable_gather(self, B, Hq, N, D, dtype, device):
        """Buffers of the transposed backward order: the layer's Q, dO, O and dQ over the whole sequence,
        [B, Hq, N, D] each (a call takes row ranges of them, so all share one set of strides), and the per-row
        statistics the dK/dV kernel reads, fp32 [2, B, Hq, N rounded up to 4]."""
        self.gather = tuple(torch.empty(B, Hq, N, D, dtype=dtype, device=device) for _ in range(4)) + (
            torch.empty(2, B, Hq, (N + 3) // 4 * 4, dtype=torch.float32, device=device),)


class ChunkAttention(torch.autograd.Function):
    """Attention of one chunk against a layer's cache; backward deposits into the layer's KV-gradient buffers."""

    @staticmethod
    def forward(ctx, q, k_new, v_new, state, q_start, scale, weights, weight_chunk_len, keep, dq_weights=None,
                rope_base=None):
        # keep: None = always compute; "store" = stage 1, remember (O, LSE); "reuse" = stage 2, take them back
        # (the rebuilt chunk has the same inputs and the kernels are deterministic, so the values are identical and
        # the cache rows already hold this chunk's K/V)
        if keep == "reuse":
            # the span of stage 1 that holds this chunk's rows (the chunk itself, or a longer span to cut from)
            s0, (o_all, lse_all) = max((kv for kv in state.kept.items() if kv[0] <= q_start), key=lambda kv: kv[0])
            a, b = q_start - s0, q_start - s0 + q.shape[2]
            if a == 0 and b == o_all.shape[2]:
                o, lse = o_all, lse_all
            else:
                o, lse = o_all[:, :, a:b].contiguous(), lse_all[:, :, a:b].contiguous()
        else:
            _b.kv_append(k_new, v_new, state.k, state.v, q_start, rope_base=rope_base)   # keys are cached rotated
            o, lse = _b.seco_chunk_attn_fwd(q, state.k, state.v, q_start, scale,
                                            o=torch.empty(q.shape, dtype=q.dtype, device=q.device))
            if keep == "store":
                state.kept[q_start] = (o, lse)
        ctx.save_for_backward(q, o, lse)
        ctx.state, ctx.q_start, ctx.scale, ctx.weights, ctx.wlen = state, q_start, scale, weights, weight_chunk_len
        ctx.dq_weights, ctx.rope_base = dq_weights, rope_base
        return o

    @staticmethod
    def backward(ctx, d_o):
        q, o, lse = ctx.saved_tensors
        st, s0, C = ctx.state, ctx.q_start, q.shape[2]
        d_o = d_o.contiguous()
        if st.gather is not None:
            # transposed order (Alg. 1 only): this chunk's finished gK/gV rows from its own and every later chunk's
            # query rows, whose Q and dO the layer has kept; nothing is added to earlier rows
            q_all, do_all, o_all, dq_all, stats = st.gather
            q_all[:, :, s0:s0 + C] = q
            do_all[:, :, s0:s0 + C] = d_o
            o_all[:, :, s0:s0 + C] = o
            row_w, wlen = None, None
            if st.gather_rows is not None:      # Alg. 2: 1 on the chunk's own rows, the factor on later selected chunks
                sel, factor, wlen, k = st.gather_rows
                j = s0 // wlen
                row_w = _b.spaco_gather_row_weights(sel, j, k, factor)
            d_q = _b.seco_chunk_attn_bwd_gather(q_all[:, :, s0:], st.k, st.v, o_all[:, :, s0:s0 + C], lse,
                                                do_all[:, :, s0:], st.gk, st.gv, s0, ctx.scale, C, stats,
                                                d_q=dq_all[:, :, s0:s0 + C], row_weight=row_w,
                                                weight_chunk_len=wlen).contiguous()
        elif ctx.weights is None and ctx.dq_weights is None:
            d_q = _b.seco_chunk_attn_bwd(q, st.k, st.v, o, lse, d_o, st.gk, st.gv, s0, ctx.scale)
        else:
            n_chunks = len(ctx.dq_weights) if ctx.weights is None else len(ctx.weights)
            w = [1.0] * n_chunks if ctx.weights is None else ctx.weights
            d_q = _b.spaco_chunk_attn_bwd(q, st.k, st.v, o, lse, d_o, st.gk, st.gv, s0, ctx.scale,
                                          w, ctx.wlen, dq_weight=ctx.dq_weights)
        d_k, d_v = _b.kvgrad_readout(st.gk, st.gv, s0, C, q.dtype, rope_base=ctx.rope_base)
        return d_q, d_k, d_v, None, None, None, None, None, None, None, None


class Rope(torch.autograd.Function):
    """Rotary position embedding of the chunk's queries (rope_rotate); the gradient is turned back."""

    @staticmethod
    def forward(ctx, x, pos_start, base):
        ctx.pos_start, ctx.base = pos_start, base
        return _b.rope_rotate(x.contiguous(), pos_start, base)

    @staticmethod
    def backward(ctx, d_out):
        return _b.rope_rotate(d_out.contiguous(), ctx.pos_start, ctx.base, inverse=True), None, None


def hand_over(params, grads):
    """Leaves every parameter's gradient in .grad (None there if no chunk reached it) and returns {name: gradient}, zeros
    for those.  A tensor under several names gets the sum over them.  A parameter that something waits for (hooks of
    the tensor, post-accumulate hooks, hooks of its accumulation node) receives its gradient through autograd, which
    runs them: once per step, with the step's gradient.
    So does a parameter that is computed from others."""
    has_grad_hooks = (_b._ext or _b._load_ext()).has_grad_hooks
    total = {}                                  # id -> gradient
    for n, t in params.items():
        g = grads.get(n)
        if g is not None and t.requires_grad:
            total[id(t)] = total[id(t)] + g if id(t) in total else g
    done = set()
    for t in params.values():
        g = total.get(id(t))
        if g is None or id(t) in done:
            continue
        done.add(id(t))
        if t.is_leaf and not has_grad_hooks(t):
            t.grad = g
        else:
            torch.autograd.backward(t, g)
    out = {}
    for n, t in params.items():
        g = total.get(id(t))
        if g is not None and t.is_leaf:
            g = t.grad                          # (a hook may have changed or taken it)
        out[n] = torch.zeros_like(t) if g is None else g
    return out


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
        relay factor `factor`).  Returns (sum of the chunk losses, as stage 1 runs them, {name: gradient}).

        The derivatives are written out, not recorded: hooks of the parameters run once per step, with its gradient
        (hand_over), not once per chunk, and saved-tensor hooks have nothing to see.

        Negative tokens count from the end of the embedding table.  A token outside it raises IndexError when the step is through,
        and no parameter receives a gradient; a target outside the head's columns (other than -100, which is left out) makes the
        loss and the gradients NaN.

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
            # stage 2 rebuilds every chunk as stage 1 ran it, launch for launch: the losses come from there, and stage 1 ends
            # at the last layer's cache rows (of a two-layer step over 4096 tokens an eighth of the time, mostly that
            # layer's attention and MLP, the final norm and the head)
            rebuilt = c1 == chunk_len and set(order) == set(range(len(starts)))
            # ... and stage 2 starts with the last chunk, whose cache rows no other chunk reads: it is run once, there, and stage 1
            # ends in front of it (4096 tokens in 8 chunks 3.79 -> 3.71 ms; two selected of 1152 in 6 chunks 1.38 -> 1.28, of 3584 in 3 2.06 -> 1.83)
            once = len(starts) - 1 if c1 == chunk_len and len(order) > 0 and order[0] == len(starts) - 1 else None
            for s0 in range(0, N if once is None else starts[once], c1):    # stage 1: inference over all chunks
                ext.step_infer(run, tokens, targets, s0, min(s0 + c1, N), None if rebuilt else losses, keep_attention_outputs)
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
                ext.step_train(run, tokens, targets, starts[j], min(starts[j] + chunk_len, N), keep_attention_outputs and j != once, w,
                               chunk_len, wq, losses if rebuilt or j == once else None)
            # (everything is on its way before the host waits for the loss)
            result, grads = ext.step_result(run), dict(zip(names, ext.step_grads(run)))
            torch.sum(losses, 0, out=result[0])
            total, outside = result.tolist()
        if outside:
            raise IndexError("tokens: an index is out of range of the embedding table")
        return total, hand_over(p, grads)
