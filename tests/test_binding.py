"""What the Python calls refuse before anything reaches the library, and how (no GPU)."""
import numpy as np
import pytest


def test_a_forked_process_is_refused(monkeypatch):
    """A child forked from a process that has used the GPU holds its tensors and cannot use them."""
    import torch
    from paper_2506_03887_amd import binding
    binding.load()
    monkeypatch.setattr(binding, "_current_device", lambda: 0)
    monkeypatch.setattr(binding, "_current_stream", lambda device: 0)
    assert binding._stream_ptr(None) == 0
    monkeypatch.setattr(binding, "_in_bad_fork", lambda: True, raising=False)
    monkeypatch.setattr(torch.cuda, "_is_in_bad_fork", lambda: True)
    with pytest.raises(RuntimeError, match="forked"):
        binding._stream_ptr(None)


@pytest.mark.parametrize("call", ["advance_fill_apply_mask", "advance_fill_argmax"])
def test_arguments_of_the_step_calls(call):
    """A bitmask without columns, rows that do not match, strided logits, host tensors: the errors that all calls raise."""
    import torch
    from paper_2506_03887_amd import Pre3
    lib = Pre3("S ::= S X | X\nX ::= [a-e]\n", np.frombuffer(b"abcde\0", np.uint8), np.arange(7), 5, stack_cap=8, host_only=True)
    tokens, mask = torch.zeros(3, dtype=torch.int32), torch.zeros((3, lib.words), dtype=torch.int32)
    logits = torch.zeros((3, 8), dtype=torch.bfloat16)
    more = (tokens,) if call == "advance_fill_argmax" else ()
    step = getattr(lib, call)
    for bad_mask, bad_logits, error in [(mask[:, 0].contiguous(), logits, IndexError), (mask.expand(3, 2).contiguous(), logits, AssertionError),
                                        (mask, logits[:2], AssertionError), (mask, logits.t().contiguous().t(), AssertionError),
                                        (mask, logits[0], AssertionError), (mask, logits, TypeError)]:
        with pytest.raises(error):
            step(tokens, bad_mask, bad_logits, *more)
