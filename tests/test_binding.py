"""What the Python calls refuse before anything reaches the library, and how (no GPU)."""
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
