"""The greedy step of more rows than compute units on long rows: two blocks share a unit, each holds the first 61,440 tokens of
its row and streams the rest.  Lockstep with the oracle, the best token on either side of every edge of that split.  And the
one-kernel form on long rows that start at any logit."""
import numpy as np
import pytest

from oracle import Oracle, masked_argmax as oracle_masked_argmax
from workloads import grammars as G
from workloads.vocab import BASE_SEED, Vocab, bf16_logits, bpe_like_vocab

pytestmark = pytest.mark.gpu

HELD = 8 * 960 * 8                         # tokens a block holds in registers


def _vocab(n):
    deep = [b"[" * 32, b"{\"k\":" * 6, b"[" * 9 + b"]" * 9, b"]" * 20, b"[1," * 10]
    return Vocab(bpe_like_vocab(n - len(deep), 16, BASE_SEED + n).tokens[:-1] + deep + [b""], n - 1)


@pytest.mark.parametrize("V,B,options,form", [
    (HELD - 1, 257, {}, "two calls"), (HELD, 257, {}, "one kernel"), (HELD + 5, 300, {}, "one kernel"),
    (HELD + 8 * 960, 258, {}, "one kernel"), (HELD + 8 * 960 * 4 + 8, 270, dict(compact_cycles=True), "one kernel"),
    (70_001, 300, dict(row_threshold=64), "one kernel"), (65_007, 257, dict(max_condition_depth=3), "one kernel"),
    (HELD + 16, 513, {}, "two calls"), (2 * HELD + 3, 520, {}, "one kernel")])
def test_greedy_step_of_more_rows_than_units(V, B, options, form):
    _lockstep(V, B, options, form, -V % 8, 0)


# (beyond four blocks of 8,192 tokens to a unit, where the spread form does not serve, on rows of 76,808 tokens and more; beyond
# 130,567 tokens, where 64 rows take 20.0 us against 16.6 to 17.5 in two calls, from a third of the units on)
@pytest.mark.parametrize("V,B,pad,offset,options,form", [
    (76_807, 200, 0, 0, {}, "two calls"), (76_809, 200, 0, 0, {}, "one kernel"), (80_001, 256, 0, 1, {}, "one kernel"),
    (100_003, 79, 4, 3, {}, "one kernel"), (100_003, 78, 4, 3, {}, "spread"), (100_003, 100, 5, 5, dict(compact_cycles=True), "one kernel"),
    (78_000, 150, 1, 0, dict(max_condition_depth=3), "one kernel"), (153_607, 86, 0, 2, {}, "one kernel"), (153_608, 86, 4, 0, {}, "two calls"),
    (130_567, 65, 0, 1, {}, "one kernel"), (130_569, 85, 0, 0, {}, "two calls"), (130_569, 86, 0, 0, {}, "one kernel"), (153_607, 64, 0, 2, {}, "two calls"),
    (100_000, 257, 1, 0, {}, "two calls")])
def test_greedy_step_on_rows_at_any_offset(V, B, pad, offset, options, form):
    _lockstep(V, B, options, form, pad, offset)


# Rows that no block holds whole, up to the longest: those of the largest vocabulary with token-level edges, and those whose mask
# row leaves room for a staged stack of 1,024 and 4,096 entries beside it (one mask word more is the two calls).
@pytest.mark.parametrize("V,B,cap,options,form", [
    (153_611, 257, 48, {}, "one kernel"), (200_003, 259, 1024, dict(compact_cycles=True), "one kernel"),
    (344_064, 257, 4096, dict(compact_cycles=True), "one kernel"), (344_065, 257, 4096, dict(compact_cycles=True), "two calls"),
    (458_750, 257, 48, {}, "one kernel"), (458_753, 257, 48, {}, "two calls")])
def test_greedy_step_on_rows_longer_than_a_unit_holds(V, B, cap, options, form):
    _lockstep(V, B, options, form, -V % 8, 0, cap, 2)


def _lockstep(V, B, options, form, pad, offset, cap=48, steps=4):
    import torch
    from paper_2506_03887_amd import Pre3
    dev = torch.device("cuda:0")
    if torch.cuda.get_device_properties(0).multi_processor_count != 256:
        pytest.skip("the lines of the dispatch are drawn for 256 compute units")
    v = _vocab(V)
    cycles = "compact_cycles" in options
    text = G.JSON_RIGHT_RECURSIVE if cycles else G.JSON
    o = Oracle(text, compact_cycles=cycles)
    lib = Pre3(text, v.bytes, v.offsets, v.eos_id, max_token_len=v.max_len, stack_cap=cap, **options)
    rng = np.random.default_rng(V + B)
    states, length, data = np.full(B, o.initial_state(0), np.int32), np.ones(B, np.int32), np.zeros((B, cap), np.int32)
    data[:, 0] = states
    s_d, l_d, d_d = (torch.from_numpy(x.copy()).to(dev) for x in (states, length, data))
    err_d, tok_d = torch.zeros(B, dtype=torch.int32, device=dev), torch.full((B,), -1, dtype=torch.int32, device=dev)
    lib.bind_state(s_d, d_d, l_d, err_d)
    mask_d = torch.zeros((B, v.words), dtype=torch.int32, device=dev)
    stride = V + pad
    view = torch.zeros(B * stride + offset, dtype=torch.int16, device=dev)[offset:].view(B, stride).view(torch.bfloat16)
    assert lib.step_form(view, greedy=True) == form and lib.step_form(view) == ("spread" if form == "spread" else "two calls")
    assert lib.step_kernel_launches(view, greedy=True) == (form != "two calls")
    if pad or offset:
        assert not lib.step_kernel_launches(view, one_kernel=True, greedy=True) or (stride % 8 == 0 and offset % 8 == 0)
    edges = [t for t in (0, 7, 8, HELD - 8, HELD - 1, HELD, HELD + 7, HELD + 8 * 960 - 1, HELD + 8 * 960, V - V % 8 - 8, V - V % 8 - 1, V - 2)
             if 0 <= t < V]
    tokens = np.full(B, -1, np.int32)
    for s in range(steps):
        err = o.advance_batch(states, data, length, tokens, v)
        if s % 2:
            ended = (states < 0) & (tokens == v.eos_id) & (err == 0)
            states[ended], length[ended] = o.initial_state(0), 1
        mask = o.fill_mask(states, data, length, v)
        host = bf16_logits(rng, B, stride)
        host[0::9] = rng.choice([0x8000, 0x0000], size=host[0::9].shape)        # zeros of both signs
        host[1::9, ::2] = 0x7FC1                                                # NaN of both signs, -inf, +inf, one value
        host[2::9] = 0xFF80
        host[3::9, ::5] = 0xFFC3
        host[4::9, 1::3] = 0x7F80
        host[5::9] = 0x3F80
        host[6::9] |= 0x8000
        for b in range(7, B, 9):                                                # the largest at the edges, alone and twice
            host[b, rng.choice(edges, size=1 + b % 2, replace=False)] = 0x4300
            host[b, rng.choice(V, size=40)] = 0x4280
        view.copy_(torch.from_numpy(host.view(np.int16)).to(dev).view(torch.bfloat16))
        lib.advance_fill_argmax(tok_d, mask_d, view, tok_d, restart_on_eos=bool(s % 2))
        want = oracle_masked_argmax(host, mask, V)
        got = tok_d.cpu().numpy()
        assert (got == want).all(), (s, np.flatnonzero(got != want)[:5], got[got != want][:5], want[got != want][:5])
        assert (err_d.cpu().numpy() == err).all() and (s_d.cpu().numpy() == states).all() and (l_d.cpu().numpy() == length).all(), s
        live = np.arange(cap)[None, :] < length[:, None]
        assert (d_d.cpu().numpy()[live] == data[live]).all(), s
        assert (mask_d.cpu().numpy().view(np.uint32) == mask).all(), s
        assert (view.view(torch.int16).cpu().numpy().view(np.uint16) == host).all(), s
        # the next tokens: mostly the oracle's choice, some refused, skipped and the end of sequence
        tokens = want.copy()
        odd = rng.random(B) < 0.2
        tokens[odd] = rng.choice([-1, V + 5, v.eos_id, *range(V - 6, V - 1)], size=int(odd.sum()))
        tok_d.copy_(torch.from_numpy(tokens))
    assert lib.fault_count() == 0
