"""SeCO / SpaCO training step of a small decoder, driven through the C ABI (Alg. 1 and Alg. 2 end to end).

The attention of every layer, its backward and the whole KV-gradient relay run in the HIP library:
each layer owns a KV cache and a pair of fp32 KV-gradient buffers that live for the whole step, the
forward of a chunk is `seco_chunk_attn_fwd` against the cache, its backward is `seco_chunk_attn_bwd` /
`spaco_chunk_attn_bwd`, which deposits the chunk's dK/dV on every visible cache row, and the gradient
handed to the chunk's own recomputed K/V is simply the chunk's rows of those buffers (they hold what
the later chunks deposited plus the chunk's own diagonal block: the relay of Alg. 1, `m_i.grad <-
m'_i.grad`), read out by `kvgrad_readout`; new keys / values enter the cache through `kv_append`.  Under SpaCO the deposits on earlier selected chunks carry the compensation
factor, so a chain through p caches is scaled by factor^p (Sec. 5).

The projections and the MLP are library GEMMs; the residual adds, norms, SiLU, loss and embedding gradient around
them are row kernels of the library (decoder.hip), one launch each, and the derivatives are written out below
instead of being recorded: at the row counts of a chunk a step is bound by the number of launches and the host time
behind each (with autograd and framework operators for the row work, 27 ms for two layers over 4096 tokens in
chunks of 512, of which the GPU worked 14).  Only one chunk's activations are alive at a time, as in the paper.
There is no CPU path.

Model (fixed here so that a checker can build the same function): pre-norm decoder, RMSNorm with
eps 1e-6, grouped-query causal attention (optionally with rotary position embedding), MLP x + silu(h W1) W2, final
RMSNorm, linear head, cross-entropy summed over tokens.  Parameter names: emb, head, norm_f and
l{i}.norm1, l{i}.norm2, l{i}.wq, l{i}.wk, l{i}.wv, l{i}.wo, l{i}.w1, l{i}.w2, all stored [in, out].
"""
from __future__ import annotations

import torch

from . import binding as _b

_GAIN_BLOCKS = 256        # partial sums of a norm gain's gradient (DEC_GAIN_BLOCKS)


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


class ChunkedDecoder:
    """Holds the parameters (dict name -> leaf tensor on the GPU) and runs SeCO / SpaCO steps."""

    def __init__(self, params, n_layers, n_q_heads, n_kv_heads, head_dim, rope_base=None):
        self.p = params
        self.rope_base = rope_base      # rotary embedding of queries and keys (keys are cached rotated), or None
        self.n_layers, self.Hq, self.Hkv, self.D = n_layers, n_q_heads, n_kv_heads, head_dim
        self.scale = float(head_dim) ** -0.5
        _b.load_library()          # fail here, loudly, if the HIP library has not been built

    def _heads(self, t, B, C):
        """[B*C, (Hq + 2 Hkv) D] rows seen as query, key and value heads, [B, H, C, D] each."""
        v = t.view(B, C, self.Hq + 2 * self.Hkv, self.D).transpose(1, 2)
        return v[:, :self.Hq], v[:, self.Hq:self.Hq + self.Hkv], v[:, self.Hq + self.Hkv:]

    def _attention(self, st, q, k, v, q_start, keep):
        """O ([B, H, C, D] view of contiguous [B, C, H, D] rows) and LSE of the chunk; k / v enter the cache.
        keep: None = always compute; "store" = stage 1, remember (O, LSE); "reuse" = stage 2, take them back (the
        rebuilt chunk has the same inputs and the kernels are deterministic, so the values are identical and the
        cache rows already hold this chunk's K/V)."""
        B, H, C, D = q.shape
        if keep == "reuse":
            # the span of stage 1 that holds this chunk's rows (the chunk itself, or a longer span to cut from)
            s0, (o, lse) = max((kv for kv in st.kept.items() if kv[0] <= q_start), key=lambda kv: kv[0])
            a, b = q_start - s0, q_start - s0 + C
            if a == 0 and b == o.shape[2]:
                return o, lse
            o = o.transpose(1, 2)[:, a:b].reshape(B * C, H * D).view(B, C, H, D).transpose(1, 2)
            return o, lse[:, :, a:b].contiguous()
        _b.kv_append(k, v, st.k, st.v, q_start, rope_base=self.rope_base)   # keys are cached rotated
        o = torch.empty(B, C, H, D, dtype=q.dtype, device=q.device).transpose(1, 2)
        _, lse = _b.seco_chunk_attn_fwd(q, st.k, st.v, q_start, self.scale, o=o)
        if keep == "store":
            st.kept[q_start] = (o, lse)
        return o, lse

    def _forward(self, tokens, B, q_start, run, keep, saved):
        """Logits of one chunk (tokens: its B*C indices).  saved: list that receives what the backward needs, or None
        (stage 1: the residual stream is updated in place)."""
        p, C, ext = self.p, tokens.shape[0] // B, run.ext
        x, y = p["emb"][tokens], None
        for l in range(self.n_layers):
            x1, h1, r1 = ext.add_rmsnorm(x, y, run.gain(f"l{l}.norm1"), None if saved is not None else x)
            qkv = torch.mm(h1, run.wqkv[l])
            q, k, v = self._heads(qkv, B, C)
            if self.rope_base is not None:
                _b.rope_rotate(q, q_start, self.rope_base, out=q)
            o, lse = self._attention(run.states[l], q, k, v, q_start, keep)
            o2 = o.transpose(1, 2).view(B * C, self.Hq * self.D)
            y = torch.mm(o2, p[f"l{l}.wo"])
            x2, h2, r2 = ext.add_rmsnorm(x1, y, run.gain(f"l{l}.norm2"), None if saved is not None else x1)
            u = torch.mm(h2, p[f"l{l}.w1"])
            a = ext.silu(u)
            y = torch.mm(a, p[f"l{l}.w2"])
            if saved is not None:
                saved.append((x1, h1, r1, qkv, q, o, o2, lse, x2, h2, r2, u, a))
            x = x2
        x, h, r = ext.add_rmsnorm(x, y, run.gain("norm_f"), None if saved is not None else x)
        if saved is not None:
            saved.append((x, h, r))
        return torch.mm(h, p["head"])

    def _attention_bwd(self, st, q, o, lse, d_o, dq, q_start, weights, wlen, dq_weights):
        """dq (same layout as q) of the chunk; its dK/dV go to the layer's KV-gradient buffers."""
        C = q.shape[2]
        if st.gather is not None:
            # transposed order: this chunk's finished gK/gV rows from its own and every later chunk's query rows,
            # whose Q and dO the layer has kept; nothing is added to earlier rows
            q_all, do_all, o_all, dq_all, stats = st.gather
            rows = slice(q_start, q_start + C)
            q_all[:, :, rows] = q
            do_all[:, :, rows] = d_o
            o_all[:, :, rows] = o
            row_w, wl = None, None
            if st.gather_rows is not None:      # Alg. 2: 1 on the chunk's own rows, the factor on later selected chunks
                sel, factor, wl, k = st.gather_rows
                row_w = _b.spaco_gather_row_weights(sel, q_start // wl, k, factor)
            _b.seco_chunk_attn_bwd_gather(q_all[:, :, q_start:], st.k, st.v, o_all[:, :, rows], lse,
                                          do_all[:, :, q_start:], st.gk, st.gv, q_start, self.scale, C, stats,
                                          d_q=dq_all[:, :, rows], row_weight=row_w, weight_chunk_len=wl)
            dq.copy_(dq_all[:, :, rows])
        elif weights is None and dq_weights is None:
            _b.seco_chunk_attn_bwd(q, st.k, st.v, o, lse, d_o, st.gk, st.gv, q_start, self.scale, d_q=dq)
        else:
            w = [1.0] * len(dq_weights) if weights is None else weights
            _b.spaco_chunk_attn_bwd(q, st.k, st.v, o, lse, d_o, st.gk, st.gv, q_start, self.scale, w, wlen, d_q=dq,
                                    dq_weight=dq_weights)

    def _backward(self, d_logits, tokens, B, q_start, run, saved, weights, wlen, dq_weights):
        """Adds the chunk's parameter gradients to run's; d_logits: gradient of its loss at the logits."""
        p, C, ext = self.p, tokens.shape[0] // B, run.ext
        x, h, r = saved.pop()
        run.add("head", h, d_logits)
        dx = ext.rmsnorm_bwd(x, run.gain("norm_f"), r, torch.mm(d_logits, p["head"].t()), None, run.part("norm_f"))
        for l in range(self.n_layers - 1, -1, -1):
            x1, h1, r1, qkv, q, o, o2, lse, x2, h2, r2, u, a = saved.pop()
            st = run.states[l]
            run.add(f"l{l}.w2", a, dx)
            du = ext.silu_bwd(u, torch.mm(dx, p[f"l{l}.w2"].t()))
            run.add(f"l{l}.w1", h2, du)
            dx = ext.rmsnorm_bwd(x2, run.gain(f"l{l}.norm2"), r2, torch.mm(du, p[f"l{l}.w1"].t()), dx,
                                 run.part(f"l{l}.norm2"))
            run.add(f"l{l}.wo", o2, dx)
            d_o = torch.mm(dx, p[f"l{l}.wo"].t()).view(B, C, self.Hq, self.D).transpose(1, 2)
            d_qkv = torch.empty_like(qkv)
            dq, dk, dv = self._heads(d_qkv, B, C)
            self._attention_bwd(st, q, o, lse, d_o, dq, q_start, weights, wlen,
                                None if dq_weights is None else dq_weights[l])
            _b.kvgrad_readout(st.gk, st.gv, q_start, C, q.dtype, d_k=dk, d_v=dv, rope_base=self.rope_base)
            if self.rope_base is not None:
                _b.rope_rotate(dq, q_start, self.rope_base, inverse=True, out=dq)
            run.add(f"l{l}.wqkv", h1, d_qkv)
            dx = ext.rmsnorm_bwd(x1, run.gain(f"l{l}.norm1"), r1, torch.mm(d_qkv, run.wqkv[l].t()), dx,
                                 run.part(f"l{l}.norm1"))
        if p["emb"].requires_grad:
            ext.embedding_bwd(dx, tokens, run.embedding())

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
        starts = list(range(0, N, chunk_len))
        states = [LayerState(B, self.Hkv, N, self.D, dtype, dev) for _ in range(self.n_layers)]
        if transposed_backward:
            if dq_weights is not None or dtype != torch.bfloat16:
                raise ValueError("the transposed backward order takes bf16 parameters and the exact dQ")
            if selected is not None and chunk_len % 64 != 0:
                raise ValueError("Alg. 2 in the transposed order needs a chunk length that is a multiple of 64")
            for st in states:
                st.enable_gather(B, self.Hq, N, self.D, dtype, dev)
                if selected is not None:
                    st.gather_rows = ({int(i) for i in selected}, float(factor), chunk_len, len(starts))
        for t in p.values():
            t.grad = None
        c1 = stage1_chunk_len or chunk_len
        order = range(len(starts) - 1, -1, -1) if selected is None else sorted({int(i) for i in selected}, reverse=True)
        with torch.no_grad():
            run = _Run(self, states)
            tokens, targets = tokens.to(torch.int64), targets.to(torch.int64)
            losses = torch.empty(N * B, dtype=torch.float32, device=dev)        # one per token, in stage-1 order
            for s0 in range(0, N, c1):                                      # stage 1: inference over all chunks
                tok, tgt = (t[:, s0:s0 + c1].reshape(-1) for t in (tokens, targets))
                logits = self._forward(tok, B, s0, run, "store" if keep_attention_outputs else None, None)
                run.ext.cross_entropy(logits, tgt, losses[s0 * B:s0 * B + tok.shape[0]])
            for st in states:
                _b.kvgrad_zero(st.gk, st.gv)
            for j in order:                                                 # stage 2: rebuild + back-propagate
                w = None if selected is None else _b.spaco_chunk_weights(order, j, factor)
                s0 = starts[j]
                wq = None if dq_weights is None else [dq_weights(j, l) for l in range(self.n_layers)]
                tok, tgt = (t[:, s0:s0 + chunk_len].reshape(-1) for t in (tokens, targets))
                saved = []
                logits = self._forward(tok, B, s0, run, "reuse" if keep_attention_outputs else None, saved)
                run.ext.cross_entropy(logits, tgt, None)                    # logits <- gradient at the logits
                self._backward(logits, tok, B, s0, run, saved, w, chunk_len, wq)
            return float(losses.sum()), run.finish()


class _Run:
    """Gradients and derived weights of one step."""

    def __init__(self, dec, states):
        self.p, self.n_layers, self.states = dec.p, dec.n_layers, states
        self.ext = _b._ext or _b._load_ext()
        self.widths = (dec.Hq * dec.D, dec.Hkv * dec.D, dec.Hkv * dec.D)
        # one projection GEMM (and one gradient GEMM each way) for queries, keys and values instead of three
        self.wqkv = [torch.cat([dec.p[f"l{l}.{n}"] for n in ("wq", "wk", "wv")], dim=1) for l in range(dec.n_layers)]
        self.grads, self.parts, self.gains = {}, {}, {}

    def gain(self, name):
        g = self.gains.get(name)
        if g is None:
            g = self.gains[name] = self.p[name].detach().contiguous()
        return g

    def part(self, name):
        t = self.parts.get(name)
        if t is None:
            t = self.parts[name] = torch.zeros(_GAIN_BLOCKS, self.p[name].shape[0], dtype=torch.float32,
                                               device=self.p[name].device)
        return t

    def embedding(self):
        t = self.grads.get("emb")
        if t is None:
            t = self.grads["emb"] = torch.zeros_like(self.p["emb"], memory_format=torch.contiguous_format)
        return t

    def wanted(self, name):
        if name.endswith(".wqkv"):
            return any(self.p[name[:-3] + n].requires_grad for n in "qkv")
        return self.p[name].requires_grad

    def add(self, name, x, dy):
        """gradient of matrix `name` += x^T dy (accumulated in fp32 inside the GEMM, rounded once per chunk)"""
        if not self.wanted(name):
            return
        g = self.grads.get(name)
        if g is None:
            self.grads[name] = torch.mm(x.t(), dy)
        else:
            g.addmm_(x.t(), dy)

    def finish(self):
        """{name: gradient} of every parameter, also left in .grad (None there if no chunk reached it)."""
        for l in range(self.n_layers):
            g = self.grads.pop(f"l{l}.wqkv", None)
            if g is not None:
                for n, part in zip(("wq", "wk", "wv"), g.split(self.widths, dim=1)):
                    self.grads[f"l{l}.{n}"] = part.contiguous()
        for n, t in self.parts.items():
            self.grads[n] = t.sum(dim=0).to(self.p[n].dtype)
        out = {}
        for n, t in self.p.items():
            if n in self.grads and t.requires_grad:
                t.grad = out[n] = self.grads[n]
            else:
                out[n] = torch.zeros_like(t)
        return out
