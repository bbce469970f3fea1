"""How the training step leaves gradients at the parameters (chunk_loop.hand_over); no GPU needed."""
import torch

from paper_2505_16710_amd.chunk_loop import hand_over


def _leaf(v=0.0):
    return torch.full((3,), v, requires_grad=True)


def test_plain_parameters_take_the_gradient_itself():
    a, b, frozen, idle = _leaf(), _leaf(), torch.zeros(3), _leaf()
    ga, gb = torch.ones(3), 2 * torch.ones(3)
    out = hand_over({"a": a, "b": b, "frozen": frozen, "idle": idle}, {"a": ga, "b": gb, "frozen": ga, "idle": None})
    assert a.grad is ga and out["a"] is ga and b.grad is gb and frozen.grad is None and idle.grad is None
    assert not out["frozen"].any() and not out["idle"].any()


def test_a_tensor_under_two_names_gets_the_sum():
    a = _leaf()
    out = hand_over({"l0.w1": a, "l1.w1": a}, {"l0.w1": torch.ones(3), "l1.w1": 2 * torch.ones(3)})
    assert torch.equal(a.grad, torch.full((3,), 3.0)) and out["l0.w1"] is a.grad and out["l1.w1"] is a.grad


def test_hooks_run_once_and_their_result_counts():
    a, b, c = _leaf(), _leaf(), _leaf()
    seen = []
    a.register_hook(lambda g: (seen.append("a"), 10 * g)[1])

    def take(t):
        seen.append("b")
        t.grad = None
    b.register_post_accumulate_grad_hook(take)
    node = c.view_as(c).grad_fn.next_functions[0][0]
    node.register_hook(lambda *_: seen.append("c"))
    g = {n: torch.ones(3) for n in "abc"}
    out = hand_over({"a": a, "b": b, "c": c}, g)
    assert sorted(seen) == ["a", "b", "c"]
    assert torch.equal(a.grad, torch.full((3,), 10.0)) and torch.equal(out["a"], a.grad)
    assert b.grad is None and not out["b"].any()
    assert torch.equal(c.grad, torch.ones(3))


def test_a_computed_parameter_passes_its_gradient_on():
    a = _leaf(1.0)
    out = hand_over({"w": 2 * a}, {"w": torch.ones(3)})
    assert torch.equal(a.grad, torch.full((3,), 2.0)) and torch.equal(out["w"], torch.ones(3))
