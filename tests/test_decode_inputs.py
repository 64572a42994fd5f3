"""BlockDecodeLoop.set_step_inputs on the CPU (host tensors throughout; nothing is run): where a step's inputs go."""
import pytest
import torch

from paper_2511_15927_amd import synth
from paper_2511_15927_amd.decode import BlockDecodeLoop


@pytest.fixture()
def loop():
    cfg = synth.mixer_cfg(2, 8, 12, d_state=4)
    params = [(synth.make_params(cfg, 1, 0), synth.make_params(cfg, 1, 1))]
    return BlockDecodeLoop(cfg, params, 2, device="cpu")


def tokens(loop, seed):
    return {k: v.to(torch.bfloat16) for k, v in synth.make_inputs(loop.cfg, seed).items()}


@pytest.mark.parametrize("kind", ["plain", "float32", "own views"])
def test_a_steps_inputs_are_what_was_given(loop, kind):
    for step in (0, 1):
        given = tokens(loop, step)
        if kind == "float32":
            given = {k: v.float() for k, v in given.items()}
        elif kind == "own views":       # parts of the step's own buffer
            loop.set_step_inputs(step, given)
            given = {k: v.clone() for k, v in loop.step_inputs[step].items()}
            loop.set_step_inputs(step, loop.step_inputs[step])
        loop.set_step_inputs(step, given)
        for k, t in loop.step_inputs[step].items():
            assert torch.equal(t, given[k].reshape(t.shape).to(t.dtype)), (step, k)


@pytest.mark.parametrize("replaced", [("x",), ("dt", "C"), ("x", "z", "dt", "B", "C")])
def test_a_tensor_that_the_caller_put_there_is_written(loop, replaced):
    """step_inputs is the caller's to read and to fill: the calls take what stands in it, so it is what is written."""
    before = {k: t.clone() for k, t in loop.step_inputs[1].items()}
    for k in replaced:
        loop.step_inputs[0][k] = torch.zeros_like(loop.step_inputs[0][k])
    given = tokens(loop, 3)
    loop.set_step_inputs(0, given)
    for k, t in loop.step_inputs[0].items():
        assert torch.equal(t, given[k].reshape(t.shape)), k
    assert all(torch.equal(t, loop.step_inputs[1][k]) for k, t in before.items())
