"""The whole step of a small batch, whose rows are spread over several blocks (each advances for itself, the last to
arrive stores): lockstep with the oracle over every way a row can come about."""
import numpy as np
import pytest

from oracle import Oracle, apply_mask as oracle_apply_mask, masked_argmax as oracle_masked_argmax
from workloads import grammars as G
from workloads.vocab import BASE_SEED, Vocab, bf16_logits, bpe_like_vocab

pytestmark = pytest.mark.gpu


def _torch():
    import torch
    return torch, torch.device("cuda:0")


def _vocab(n):
    """n tokens, the last one the end of sequence; some nest deep enough to spill the walk's private stack."""
    deep = [b"[" * 32, b"[" * 17 + b"1", b"{\"k\":" * 6, b"[" * 9 + b"]" * 9, b"", b"]" * 20, b"[1," * 10, b"]]]]]]]],"]
    base = bpe_like_vocab(n - len(deep), 16, BASE_SEED + n).tokens[:-1]
    return Vocab(base + deep + [b""], n - 1)


# the number of blocks per row changes at 8,192 tokens
@pytest.mark.parametrize("greedy", [False, True])
@pytest.mark.parametrize("V,B,pad,offset,options", [
    (600, 5, 0, 0, {}), (8191, 3, 0, 1, {}), (8192, 4, 0, 0, {}), (8193, 4, 0, 0, {}), (20_003, 30, 0, 0, {}), (20_003, 8, 5, 3, {}),
    (16_392, 9, 0, 0, dict(max_condition_depth=3)), (3003, 70, 0, 0, dict(max_condition_depth=2)),
    (12_000, 12, 8, 0, dict(token_effects=False)), (9001, 6, 0, 0, dict(row_threshold=64)),
    (16_777, 10, 0, 0, dict(compact_cycles=True)), (1001, 300, 0, 0, {}), (65_003, 100, 0, 0, {}), (65_003, 130, 0, 0, {}),
    (24_577, 6, 3, 1, dict(max_condition_depth=2)), (16_392, 9, 0, 0, dict(compact_cycles=True, max_condition_depth=3))])
def test_spread_step_in_lockstep_with_the_oracle(V, B, pad, offset, options, greedy):
    """Allowed, refused, skipped, out-of-range and EOS tokens, overflow of a small stack, finished rows and restarts;
    masked logits with what lies around the rows, or the greedy choice on special rows fed back as the next token
    (the token buffer updated in place).  70 x 3,003 and 300 x 1,001 have a block per row, 130 x 65,003 exceeds four
    blocks per compute unit (the two calls), row_threshold keeps id lists (the two calls); a depth of 2 or 3 entries leaves
    tokens and whole rows open."""
    from paper_2506_03887_amd import Pre3
    torch, dev = _torch()
    v = _vocab(V)
    cycles = options.get("compact_cycles", False)
    grammar = G.JSON_RIGHT_RECURSIVE if cycles else G.JSON
    o = Oracle(grammar, compact_cycles=cycles)
    cap, W = 48, v.words
    lib = Pre3(grammar, v.bytes, v.offsets, v.eos_id, max_token_len=max(1, v.max_len), stack_cap=64, **options)
    rng = np.random.default_rng(V + B + greedy)
    s0 = o.initial_state(0)
    states, length, data = np.full(B, s0, np.int32), np.ones(B, np.int32), np.zeros((B, cap), np.int32)
    data[:, 0] = s0
    s_d, l_d, d_d = (torch.from_numpy(x.copy()).to(dev) for x in (states, length, data))
    err_d = torch.zeros(B, dtype=torch.int32, device=dev)
    lib.bind_state(s_d, d_d, l_d, err_d)
    mask_d = torch.zeros((B, W), dtype=torch.int32, device=dev)
    stride = V + pad
    flat = torch.full((B * stride + offset + 16,), 0x2345, dtype=torch.int16, device=dev)
    view = flat[offset: offset + B * stride].view(B, stride)
    tok_d = torch.zeros(B, dtype=torch.int32, device=dev)
    spread = "row_threshold" not in options and B * -(-V // 8192) <= 4 * torch.cuda.get_device_properties(0).multi_processor_count
    assert lib.step_form(view, greedy=greedy) == ("spread" if spread else "two calls")
    tokens = None
    for s in range(14):
        mask = o.fill_mask(states, data, length, v)
        if tokens is None or not greedy:
            # mostly allowed tokens, some of the deep ones, and every kind that is refused or skipped
            tokens = np.zeros(B, np.int32)
            for b in range(B):
                ids = np.flatnonzero((mask[b][np.arange(V) >> 5] >> (np.arange(V) & 31).astype(np.uint32)) & 1)
                tokens[b] = rng.choice(ids) if len(ids) else v.eos_id
            odd = rng.random(B) < 0.3
            tokens[odd] = rng.choice([-1, V + 5, v.eos_id, *range(V - 9, V - 1), *rng.integers(0, V, 6)], size=int(odd.sum()))
            tok_d.copy_(torch.from_numpy(tokens))
        restart = s % 3 != 0
        err = o.advance_batch(states, data, length, tokens, v)
        if restart:
            ended = (states < 0) & (tokens == v.eos_id) & (err == 0)
            states[ended], length[ended] = s0, 1
        want_mask = o.fill_mask(states, data, length, v)
        host = bf16_logits(rng, B, stride)
        if greedy:
            host[0::7, :V] = np.where(rng.random((len(host[0::7]), V)) < 0.5, 0x8000, 0x0000)    # zeros of both signs
            host[1::7, :V:2] = 0x7FC1                                                            # NaN, infinities
            host[2::7, :V] = 0xFF80
            host[3::7, :V:5] = 0xFFC1
        else:
            host[:, V:] = 0x1234
        view.copy_(torch.from_numpy(host.view(np.int16)).to(dev))
        if greedy:
            lib.advance_fill_argmax(tok_d, mask_d, view.view(torch.bfloat16), tok_d, restart_on_eos=restart)
            assert (view.cpu().numpy().view(np.uint16) == host).all()
            tokens = oracle_masked_argmax(np.ascontiguousarray(host), want_mask, V)
            assert (tok_d.cpu().numpy() == tokens).all(), s
        else:
            lib.advance_fill_apply_mask(tok_d, mask_d, view.view(torch.bfloat16), restart_on_eos=restart)
            oracle_apply_mask(host, want_mask, V)
            assert (view.cpu().numpy().view(np.uint16) == host).all(), s
        assert (err_d.cpu().numpy() == err).all(), s
        assert (s_d.cpu().numpy() == states).all() and (l_d.cpu().numpy() == length).all(), s
        live = np.arange(cap)[None, :] < length[:, None]
        assert (d_d.cpu().numpy()[live] == data[live]).all(), s
        assert (mask_d.cpu().numpy().view(np.uint32) == want_mask).all(), s
        assert (flat[:offset] == 0x2345).all() and (flat[offset + B * stride:] == 0x2345).all()


def test_spread_step_after_rebinding_and_in_a_graph():
    """Batches that grow and shrink on one handle, then a captured step replayed with other tokens and logits in
    between: the counters that the blocks of a row meet at are back at zero after every launch."""
    from paper_2506_03887_amd import Pre3
    torch, dev = _torch()
    v = _vocab(20_003)
    o = Oracle(G.JSON)
    lib = Pre3(G.JSON, v.bytes, v.offsets, v.eos_id, max_token_len=max(1, v.max_len), stack_cap=64)
    rng = np.random.default_rng(5)
    for B in (3, 200, 7, 40):
        states, length, data = np.full(B, o.initial_state(0), np.int32), np.ones(B, np.int32), np.zeros((B, 64), np.int32)
        data[:, 0] = states
        s_d, l_d, d_d = (torch.from_numpy(x.copy()).to(dev) for x in (states, length, data))
        err_d, tok_d = torch.zeros(B, dtype=torch.int32, device=dev), torch.zeros(B, dtype=torch.int32, device=dev)
        mask_d = torch.zeros((B, v.words), dtype=torch.int32, device=dev)
        logits = torch.zeros((B, v.n_tokens), dtype=torch.bfloat16, device=dev)
        lib.bind_state(s_d, d_d, l_d, err_d)
        graph = None
        tokens = np.full(B, -1, np.int32)
        for s in range(6):
            host = bf16_logits(rng, B, v.n_tokens)
            logits.copy_(torch.from_numpy(host.view(np.int16)).to(dev).view(torch.bfloat16))
            o.advance_batch(states, data, length, tokens, v)
            want = oracle_masked_argmax(host, o.fill_mask(states, data, length, v), v.n_tokens)
            tok_d.copy_(torch.from_numpy(tokens))
            if s < 2:
                lib.advance_fill_argmax(tok_d, mask_d, logits, tok_d)
            else:
                if graph is None:
                    graph = torch.cuda.CUDAGraph()
                    torch.cuda.synchronize()
                    with torch.cuda.graph(graph):
                        lib.advance_fill_argmax(tok_d, mask_d, logits, tok_d)
                graph.replay()
            torch.cuda.synchronize()
            assert (tok_d.cpu().numpy() == want).all(), (B, s)
            tokens = want


@pytest.mark.parametrize("B,V,cycles", [(513, 2003, False), (700, 40_001, False), (1100, 2003, False), (1100, 2003, True), (1030, 33_000, False)])
def test_advance_and_mask_of_large_batches(B, V, cycles):
    """pre3_advance_fill_mask on batches whose kernel runs with fewer threads per sequence (more than two blocks of
    512 to a compute unit; two waves for large batches of short rows): allowed, refused, skipped and EOS tokens."""
    from paper_2506_03887_amd import Pre3
    torch, dev = _torch()
    v = _vocab(V)
    grammar = G.JSON_RIGHT_RECURSIVE if cycles else G.JSON
    o = Oracle(grammar, compact_cycles=cycles)
    lib = Pre3(grammar, v.bytes, v.offsets, v.eos_id, max_token_len=max(1, v.max_len), stack_cap=48, compact_cycles=cycles)
    rng = np.random.default_rng(B)
    states, length, data = np.full(B, o.initial_state(0), np.int32), np.ones(B, np.int32), np.zeros((B, 48), np.int32)
    data[:, 0] = states
    s_d, l_d, d_d = (torch.from_numpy(x.copy()).to(dev) for x in (states, length, data))
    err_d, tok_d = torch.zeros(B, dtype=torch.int32, device=dev), torch.zeros(B, dtype=torch.int32, device=dev)
    mask_d = torch.zeros((B, v.words), dtype=torch.int32, device=dev)
    lib.bind_state(s_d, d_d, l_d, err_d)
    mask = o.fill_mask(states, data, length, v)
    for s in range(4):
        tokens = np.array([rng.choice(np.flatnonzero((m[np.arange(V) >> 5] >> (np.arange(V) & 31).astype(np.uint32)) & 1))
                           if m.any() else v.eos_id for m in mask], dtype=np.int32)
        odd = rng.random(B) < 0.2
        tokens[odd] = rng.choice([-1, V + 5, v.eos_id, *range(V - 9, V - 1)], size=int(odd.sum()))
        tok_d.copy_(torch.from_numpy(tokens))
        err = o.advance_batch(states, data, length, tokens, v)
        mask = o.fill_mask(states, data, length, v)
        lib.advance_fill_mask(tok_d, mask_d)
        assert (err_d.cpu().numpy() == err).all() and (s_d.cpu().numpy() == states).all() and (l_d.cpu().numpy() == length).all(), s
        live = np.arange(48)[None, :] < length[:, None]
        assert (d_d.cpu().numpy()[live] == data[live]).all(), s
        assert (mask_d.cpu().numpy().view(np.uint32) == mask).all(), s
