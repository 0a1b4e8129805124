"""The stack a wave walks in its registers: 64 entries of the window and 64 pushed states, everything beyond in memory.
Tokens that push and pop 63, 64, 65 and more states, from stacks of 1 to 200 entries, through every call that advances by
tokens, and forced bytes that do so through jump_forward."""
import numpy as np
import pytest

from oracle import Oracle, apply_mask as oracle_apply_mask, masked_argmax as oracle_masked_argmax
from workloads import grammars as G
from workloads.vocab import BASE_SEED, Vocab, bf16_logits, bpe_like_vocab

pytestmark = pytest.mark.gpu

DEEP = [b"[" * n for n in (15, 16, 17, 31, 32, 63, 64, 65, 66, 128, 130)] + [b"]" * n for n in (16, 62, 63, 64, 65, 66, 130)] + \
       [b"[" * 70 + b"]" * 69, b"]" * 60 + b",[", b"1" + b"]" * 63, b"1" + b"]" * 64 + b",", b"[1," * 40, b"{\"k\":" * 23, b" " * 70 + b"[" * 60]
CALLS = ("advance", "advance_fill", "step", "one_kernel", "greedy", "greedy_one_kernel")


@pytest.mark.parametrize("options", [{}, dict(token_effects=False), dict(max_condition_depth=2), dict(compact_cycles=True)])
@pytest.mark.parametrize("call", CALLS)
def test_tokens_deeper_than_the_registers(call, options):
    import torch
    from paper_2506_03887_amd import Pre3
    dev = torch.device("cuda:0")
    base = bpe_like_vocab(1000, 8, BASE_SEED + 91).tokens[:-1]
    toks = base + DEEP + [b""]
    v = Vocab(toks, len(toks) - 1)
    cycles = "compact_cycles" in options
    text = G.JSON_RIGHT_RECURSIVE if cycles else G.JSON
    o = Oracle(text, compact_cycles=cycles)
    cap = 512
    lib = Pre3(text, v.bytes, v.offsets, v.eos_id, max_token_len=v.max_len, **options)
    rows = [(depth, t) for depth in (0, 1, 15, 62, 63, 64, 65, 130, 190) for t in range(len(base), len(base) + len(DEEP) + 1)]
    if call.endswith("one_kernel"):
        rows = rows[:: len(rows) // 100]            # (the form is asked for; one row per compute unit is enough)
    elif call == "greedy":
        rows = rows[::2]                            # (fewer than half a row per compute unit: the spread form)
    B = len(rows)
    data, length = np.zeros((B, cap), np.int32), np.ones(B, np.int32)
    for b, (depth, _) in enumerate(rows):
        st = o.initial_stack(0) if depth == 0 else o.advance(o.initial_stack(0), b"[" * depth)[1]
        data[b, : len(st)], length[b] = st, len(st)
    states = data[np.arange(B), length - 1].copy()
    tokens = np.array([t for _, t in rows], np.int32)
    s_d, d_d, l_d, t_d = (torch.from_numpy(x.copy()).to(dev) for x in (states, data, length, tokens))
    e_d = torch.full((B,), -5, dtype=torch.int32, device=dev)
    lib.bind_state(s_d, d_d, l_d, e_d)
    mask = torch.full((B, v.words), 0x77777777, dtype=torch.int32, device=dev)
    x = bf16_logits(np.random.default_rng(5), B, -(-v.n_tokens // 8) * 8)
    x_d = torch.from_numpy(x.view(np.int16).copy()).to(dev)
    if call == "advance":
        lib.advance(t_d)
    elif call == "advance_fill":
        lib.advance_fill_mask(t_d, mask)
    elif call.startswith("greedy"):
        assert lib.step_form(x_d, greedy=True, one_kernel=call == "greedy_one_kernel") == ("spread" if call == "greedy" else "one kernel")
        next_d = torch.full_like(t_d, -7)
        lib.advance_fill_argmax(t_d, mask, x_d.view(torch.bfloat16), next_d, one_kernel=call == "greedy_one_kernel")
    else:
        lib.advance_fill_apply_mask(t_d, mask, x_d, one_kernel=call == "one_kernel")
    s_h, d_h, l_h = states.copy(), data.copy(), length.copy()
    err = o.advance_batch(s_h, d_h, l_h, tokens, v)
    assert set(err.tolist()) >= {0, 1} and (l_h - length).max() >= (63 if not cycles else 20) and (cycles or (length - l_h).max() >= 63)
    assert (e_d.cpu().numpy() == err).all()
    assert (s_d.cpu().numpy() == s_h).all() and (l_d.cpu().numpy() == l_h).all()
    live = np.arange(cap)[None, :] < l_h[:, None]
    assert (d_d.cpu().numpy()[live] == d_h[live]).all()
    if call != "advance":
        want = o.fill_mask(s_h, d_h, l_h, v)
        assert (mask.cpu().numpy().view(np.uint32) == want).all()
        if call.startswith("greedy"):
            assert (next_d.cpu().numpy() == oracle_masked_argmax(x, want, v.n_tokens)).all()
        elif call != "advance_fill":
            oracle_apply_mask(x, want, v.n_tokens)
        assert (x_d.cpu().numpy().view(np.uint16) == x).all()
    assert lib.fault_count() == 0


@pytest.mark.parametrize("options", [{}, dict(compact_cycles=True)])
@pytest.mark.parametrize("call", ["one_kernel", "greedy_one_kernel", "step"])
def test_effect_records_of_every_length(call, options):
    """Tokens whose stack-effect records push 6 to 143 states: the lists come 16 words at a time where the advance keeps to
    scalar loads (the one-kernel forms), as one vector load elsewhere, and in parts of 64."""
    import torch
    from paper_2506_03887_amd import Pre3
    dev = torch.device("cuda:0")
    base = bpe_like_vocab(2000, 8, BASE_SEED + 95).tokens[:-1]
    new = [b"[" * n + tail for n in range(2, 71) for tail in (b"", b"1,")]
    v = Vocab(base + new + [b""], len(base) + len(new))
    cycles = "compact_cycles" in options
    text = G.JSON_RIGHT_RECURSIVE if cycles else G.JSON
    o, cap, B = Oracle(text, compact_cycles=cycles), 256, len(new)
    lib = Pre3(text, v.bytes, v.offsets, v.eos_id, max_token_len=v.max_len, stack_cap=cap, **options)
    start = o.initial_stack(0)
    pushes = {lib.debug_token_effect(start, len(base) + i)[3] for i in range(B) if lib.debug_token_effect(start, len(base) + i)}
    assert pushes >= {*range(6, 70)} and max(pushes) > 128
    data, length = np.zeros((B, cap), np.int32), np.full(B, len(start), np.int32)
    data[:, : len(start)] = start
    states, tokens = data[:, len(start) - 1].copy(), np.arange(len(base), len(base) + B, dtype=np.int32)
    s_d, d_d, l_d, t_d = (torch.from_numpy(x.copy()).to(dev) for x in (states, data, length, tokens))
    e_d, next_d = torch.full((B,), -5, dtype=torch.int32, device=dev), torch.full((B,), -7, dtype=torch.int32, device=dev)
    lib.bind_state(s_d, d_d, l_d, e_d)
    mask = torch.zeros((B, v.words), dtype=torch.int32, device=dev)
    x = bf16_logits(np.random.default_rng(6), B, -(-v.n_tokens // 8) * 8)
    x_d = torch.from_numpy(x.view(np.int16).copy()).to(dev)
    if call == "greedy_one_kernel":
        lib.advance_fill_argmax(t_d, mask, x_d.view(torch.bfloat16), next_d, one_kernel=True)
    else:
        lib.advance_fill_apply_mask(t_d, mask, x_d, one_kernel=call == "one_kernel")
    err = o.advance_batch(states, data, length, tokens, v)
    want = o.fill_mask(states, data, length, v)
    assert (err == 0).all() and (e_d.cpu().numpy() == 0).all()
    assert (s_d.cpu().numpy() == states).all() and (l_d.cpu().numpy() == length).all()
    live = np.arange(cap)[None, :] < length[:, None]
    assert (d_d.cpu().numpy()[live] == data[live]).all()
    assert (mask.cpu().numpy().view(np.uint32) == want).all()
    if call == "greedy_one_kernel":
        assert (next_d.cpu().numpy() == oracle_masked_argmax(x, want, v.n_tokens)).all()
    assert lib.fault_count() == 0


@pytest.mark.parametrize("empties", [62, 63, 64, 65, 70])
def test_forced_bytes_deeper_than_the_registers(empties):
    """One forced byte pushes `empties` states of empty nonterminals, another pops them again, and as many closing brackets as
    were opened are forced behind it: from stacks on both sides of the window, with every length of the result."""
    from test_gpu_jump_forward import _compare
    from paper_2506_03887_amd import Pre3
    text = 'S ::= "(" S ")" | "[" %s "a" "b" "]"\nE ::= ""' % " ".join(["E"] * empties)
    v = Vocab([b"(", b")", b"[", b"a", b"b", b"]", b""], 6)
    o = Oracle([text])
    cap = 384
    lib = Pre3([text], v.bytes, v.offsets, v.eos_id, stack_cap=cap)
    prefixes = [b"(" * n + tail for n in (0, 1, 2, 60, 61, 62, 63, 64, 65, 66, 127, 128, 130) for tail in (b"[", b"[a", b"[ab", b"[ab]", b"")]
    data, length = np.zeros((len(prefixes), cap), np.int32), np.ones(len(prefixes), np.int32)
    for b, p in enumerate(prefixes):
        st = o.advance(o.initial_stack(0), p)[1] if p else o.initial_stack(0)
        data[b, : len(st)], length[b] = st, len(st)
    states = data[np.arange(len(prefixes)), length - 1].copy()
    assert length.max() > 130 + empties
    for most in (1, 2, 3, 5, 64, 200):
        assert _compare(o, lib, states, data, length, most) > 0
    assert lib.fault_count() == 0
