"""What the training step refuses before it allocates or launches anything: its kernels take sizes and addresses on trust.
Every call here gets host tensors and fails (no GPU needed)."""
import pytest
import torch

from paper_2505_16710_amd import binding as B

DM, V, HQ, HKV, D, FF = 64, 40, 2, 1, 128, (96, 160, 64)
MATRICES = {"wq": (DM, HQ * D), "wk": (DM, HKV * D), "wv": (DM, HKV * D), "wo": (HQ * D, DM)}
LAYER = ("norm1", "norm2", "wq", "wk", "wv", "wo", "w1", "w2")


def _params(**replaced):
    """[emb, head, norm_f, then the layers'] as step_new takes them; replaced: l1_wo=..., head=..."""
    p = {"emb": torch.zeros(V, DM), "head": torch.zeros(DM, V), "norm_f": torch.ones(DM)}
    for l, ff in enumerate(FF):
        shapes = {"norm1": (DM,), "norm2": (DM,), **MATRICES, "w1": (DM, ff), "w2": (ff, DM)}
        p.update({f"l{l}_{n}": torch.zeros(shapes[n]) for n in LAYER})
    p = {n: t.to(torch.bfloat16) for n, t in p.items()}
    assert set(replaced) <= set(p)
    p.update(replaced)
    return list(p.values())


def _new(params, layers=3, tokens=64, chunk=32):
    ext = B._ext or B._load_ext()
    return ext.step_new((layers, HQ, HKV, D, D ** -0.5, None, 1, tokens, chunk, chunk, False), params)


@pytest.mark.parametrize("name,shape", [
    ("l1_wo", (HQ * D, DM + 8)), ("l1_wo", (HQ * D - 8, DM)), ("l2_w2", (FF[2], DM - 8)), ("l2_w2", (FF[2] + 8, DM)),
    ("l0_w1", (DM + 8, FF[0])), ("l1_w1", (DM, FF[1] + 8)), ("l1_wq", (DM, HQ * D + 8)), ("l1_wk", (DM, HKV * D - 8)),
    ("l0_wv", (DM - 8, HKV * D)), ("head", (DM + 8, V)), ("head", (DM,)), ("emb", (V, DM, 1)), ("emb", (V, DM - 8)),
    ("l0_wq", (1, DM, HQ * D)), ("head", (DM, 0)), ("emb", (V, 0)),
])
def test_matrices_of_another_shape_are_refused(name, shape):
    with pytest.raises(ValueError, match="shape of"):
        _new(_params(**{name: torch.zeros(shape, dtype=torch.bfloat16)}))


def test_projections_whose_widths_only_add_up_are_refused():
    """wq narrower and wk wider by as much: the joint projection has the right width, its columns the wrong meaning."""
    with pytest.raises(ValueError, match="shape of wq"):
        _new(_params(l1_wq=torch.zeros(DM, HQ * D - 8, dtype=torch.bfloat16),
                     l1_wk=torch.zeros(DM, HKV * D + 8, dtype=torch.bfloat16)))


def test_sizes_that_are_not_positive_are_refused():
    with pytest.raises(ValueError, match="positive"):
        _new(_params(), chunk=0)
    with pytest.raises(ValueError, match="positive"):
        _new(_params(), tokens=0)
    with pytest.raises(ValueError, match="number of parameters"):
        _new(_params()[:-1])


@pytest.mark.parametrize("name", ["l1_norm1", "l2_norm2", "norm_f"])
@pytest.mark.parametrize("shape", [(DM - 1,), (DM + 8,), (2, DM), (DM, 1), (0,)])
def test_gains_of_another_shape_are_refused(name, shape):
    with pytest.raises(ValueError, match="shape of"):
        _new(_params(**{name: torch.ones(shape, dtype=torch.bfloat16)}))


@pytest.mark.parametrize("changed", [
    {"head": torch.float32}, {"norm_f": torch.float32}, {"l1_norm1": torch.float32}, {"l0_wo": torch.float32},
    {"l2_w2": torch.float32}, {"emb": torch.float32}, {"head": torch.float64, "norm_f": torch.float64},
    {"l1_wq": torch.float32}, {"l1_wv": torch.float32},
])
def test_dtypes_that_the_products_cannot_mix_are_refused(changed):
    names = ["emb", "head", "norm_f"] + [f"l{l}_{n}" for l in range(3) for n in LAYER]
    p = dict(zip(names, _params()))
    with pytest.raises(TypeError):
        _new(_params(**{n: p[n].to(dt) for n, dt in changed.items()}))


def test_host_tensors_are_refused():
    """Parameters that are in order otherwise (the refusals above are not refusals of the device)."""
    with pytest.raises(ValueError, match="on one GPU"):
        _new(_params())
    with pytest.raises(ValueError, match="on one GPU"):      # ... nor are the mixtures that are accepted
        p = _params()
        _new([p[0], p[1].float(), p[2].float()] + p[3:])


def _decoder():
    from paper_2505_16710_amd.chunk_loop import ChunkedDecoder
    names = ["emb", "head", "norm_f"] + [f"l{l}.{n}" for l in range(3) for n in LAYER]
    return ChunkedDecoder(dict(zip(names, _params())), 3, HQ, HKV, D)


@pytest.mark.parametrize("tokens,targets,error", [
    ((1, 64), (1, 63), ValueError), ((2, 64), (1, 64), ValueError), ((2, 64), (1, 128), ValueError),
    ((64,), (64,), ValueError), ((1, 64), (1, 64, 1), ValueError),
])
def test_targets_that_do_not_cover_the_tokens_are_refused(tokens, targets, error):
    with pytest.raises(error, match="not enough values|one target per token"):
        _decoder().step(torch.zeros(tokens, dtype=torch.int64), torch.zeros(targets, dtype=torch.int64), 32)


def test_tokens_and_targets_of_another_kind_are_refused():
    ints = torch.zeros(1, 64, dtype=torch.int64)
    for other in (ints.float(), ints.bool()):
        with pytest.raises(TypeError, match="integers"):
            _decoder().step(other, ints, 32)
        with pytest.raises(TypeError, match="integers"):
            _decoder().step(ints, other, 32)
    with pytest.raises(ValueError, match="device"):
        _decoder().step(ints, ints.to("meta"), 32)


def test_chunks_that_straddle_two_kept_spans_are_refused():
    ints = torch.zeros(1, 192, dtype=torch.int64)
    with pytest.raises(ValueError, match="kept attention outputs"):
        _decoder().step(ints, ints, 64, keep_attention_outputs=True, stage1_chunk_len=96)
    with pytest.raises(ValueError, match="on one GPU"):      # the chunks in use lie within one span each
        _decoder().step(ints, ints, 64, selected=[2, 0], keep_attention_outputs=True, stage1_chunk_len=96)
    with pytest.raises(ValueError, match="on one GPU"):      # not kept: the two lengths need not fit
        _decoder().step(ints, ints, 64, stage1_chunk_len=96)
