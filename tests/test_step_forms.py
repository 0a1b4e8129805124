"""Which form the one-call steps take, and what the choice has to keep to: limits of the kernels, workspaces, the answer
of the query.  The rules are host code and are called in the library without a GPU; tests marked gpu run the calls."""
import ctypes

import numpy as np
import pytest

from oracle import Oracle, masked_argmax as oracle_masked_argmax
from workloads import grammars as G
from workloads.vocab import Vocab, bf16_logits


def _rule(mangled, restype, *argtypes):
    """A rule of the library (namespace pre3) as a callable."""
    from paper_2506_03887_amd import load
    fn = getattr(load(), mangled)
    fn.restype, fn.argtypes = restype, argtypes
    return fn


def _one_kernel_fits(n_tokens, greedy):
    fits = _rule("_ZN4pre323advance_fill_apply_fitsEiiibb", ctypes.c_bool, *[ctypes.c_int] * 3, ctypes.c_bool, ctypes.c_bool)
    return fits(n_tokens, (n_tokens + 31) // 32, 64, False, greedy)


@pytest.mark.parametrize("n_tokens,greedy,masking", [(1, False, True), (5, False, True), (7, False, True), (8, True, True), (9, True, True),
                                                     (153_600, True, True), (153_608, False, True), (207_360, False, True), (207_368, False, False)])
def test_vocabularies_the_one_kernel_serves(n_tokens, greedy, masking):
    """The greedy form loads 16 bytes from the row's last whole group of 8 logits in every slot beyond the row: a
    vocabulary without a whole group has nothing it may load (the last row need not reach past its n_tokens logits)."""
    assert _one_kernel_fits(n_tokens, True) == greedy and _one_kernel_fits(n_tokens, False) == masking


def _tiny_vocab(n):
    return Vocab([b"a", b"(", b")", b"+", b"*", b"a+", b"(a", b")*", b"a)"][: n - 1] + [b""], n - 1)


@pytest.mark.gpu
@pytest.mark.parametrize("V", [2, 5, 6, 7, 8, 9])
@pytest.mark.parametrize("one_kernel", [False, True])
def test_greedy_step_on_vocabularies_of_a_few_tokens(V, one_kernel):
    """256 rows, 16-byte aligned with a stride of 8 or 16, the last of which ends with its V logits: tokens, states, masks
    against the oracle over a few steps."""
    import torch
    from paper_2506_03887_amd import Pre3
    dev = torch.device("cuda:0")
    v, o, B, cap = _tiny_vocab(V), Oracle(G.ARITHMETIC), 256, 32
    lib = Pre3(G.ARITHMETIC, v.bytes, v.offsets, v.eos_id, stack_cap=cap)
    states, length, data = np.full(B, o.initial_state(0), np.int32), np.ones(B, np.int32), np.zeros((B, cap), np.int32)
    data[:, 0] = states
    s_d, l_d, d_d = (torch.from_numpy(x.copy()).to(dev) for x in (states, length, data))
    err_d, tok_d = torch.zeros(B, dtype=torch.int32, device=dev), torch.full((B,), -1, dtype=torch.int32, device=dev)
    lib.bind_state(s_d, d_d, l_d, err_d)
    mask_d = torch.zeros((B, 1), dtype=torch.int32, device=dev)
    stride = (V + 7) // 8 * 8
    flat = torch.zeros((B - 1) * stride + V, dtype=torch.int16, device=dev)
    view = flat.as_strided((B, V), (stride, 1))
    rng, tokens = np.random.default_rng(V), np.full(B, -1, np.int32)
    for s in range(6):
        err = o.advance_batch(states, data, length, tokens, v)
        mask = o.fill_mask(states, data, length, v)
        host = bf16_logits(rng, B, V)
        view.copy_(torch.from_numpy(host.view(np.int16)).to(dev))
        lib.advance_fill_argmax(tok_d, mask_d, view.view(torch.bfloat16), tok_d, one_kernel=one_kernel)
        tokens = oracle_masked_argmax(host, mask, V)
        assert (tok_d.cpu().numpy() == tokens).all() and (err_d.cpu().numpy() == err).all(), s
        assert (s_d.cpu().numpy() == states).all() and (mask_d.cpu().numpy().view(np.uint32) == mask).all(), s
