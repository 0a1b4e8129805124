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


def _nesting_vocab(n):
    """n tokens of JSON text, the last one the end of sequence; some nest deep enough to spill a walk's private stack."""
    from workloads.vocab import BASE_SEED, bpe_like_vocab
    deep = [b"[" * 32, b"[" * 17 + b"1", b"{\"k\":" * 6, b"[" * 9 + b"]" * 9, b"[1," * 10, b"]" * 20]
    return Vocab(bpe_like_vocab(n - len(deep), 16, BASE_SEED + n).tokens[:-1] + deep + [b""], n - 1)


@pytest.mark.parametrize("V,compact", [(600, False), (8192, False), (20_003, False), (40_001, True), (128_256, False)])
def test_a_smaller_batch_never_needs_a_larger_workspace(V, compact):
    """Rebinding to fewer sequences must not replace (and free) a workspace that work recorded for the larger batch uses,
    although the smaller batch may take a form with a spill column per block or more segments per row."""
    from paper_2506_03887_amd import Pre3
    v = _nesting_vocab(V)
    lib = Pre3(G.JSON_RIGHT_RECURSIVE if compact else G.JSON, v.bytes, v.offsets, v.eos_id, max_token_len=v.max_len, stack_cap=64,
               compact_cycles=compact, host_only=True)
    assert lib.walk_depth_bound > 16
    sizes = [1, 2, 3, 7, 16, 31, 60, 64, 65, 85, 100, 128, 200, 255, 256, 257, 341, 342, 400, 512, 700, 1024, 1025, 1500, 2048, 5000]
    held = [lib.workspace_bytes(b) for b in sizes]
    for name in held[0]:
        row = [h[name] for h in held]
        assert row == sorted(row), (name, list(zip(sizes, row)))
    seg, deep = -(-V // 8192), lib.walk_depth_bound - 16
    for b, h in zip(sizes, held):                       # enough for the batch in whichever form it runs
        blocks = b * seg if b * seg <= 1024 else 0
        assert h["advance_spill"] >= 4 * deep * max(b, blocks) and h["walk_spill"] >= 4 * deep * 64 * max(b, blocks)
        assert h["step_counters"] >= 24 * b and h["argmax"] >= 8 * b         # (the top-k counts the blocks of every bound row)


@pytest.mark.gpu
def test_a_graph_of_a_larger_batch_outlives_rebinding_to_a_smaller_one():
    """400 rows (20,003 tokens: the two launches) recorded, then 200 rows bound (spread over 600 blocks, more spill columns
    than 400) and stepped: the replay on the 400 rows' buffers gives the oracle's states, stacks, masks and tokens."""
    import torch
    from paper_2506_03887_amd import Pre3
    dev = torch.device("cuda:0")
    v, o, cap = _nesting_vocab(20_003), Oracle(G.JSON), 64
    lib = Pre3(G.JSON, v.bytes, v.offsets, v.eos_id, max_token_len=v.max_len, stack_cap=cap)
    rng = np.random.default_rng(11)

    def batch(B):
        h = dict(states=np.full(B, o.initial_state(0), np.int32), length=np.ones(B, np.int32), data=np.zeros((B, cap), np.int32))
        h["data"][:, 0] = h["states"]
        d = {k: torch.from_numpy(x.copy()).to(dev) for k, x in h.items()}
        d.update(err=torch.zeros(B, dtype=torch.int32, device=dev), tok=torch.full((B,), -1, dtype=torch.int32, device=dev),
                 mask=torch.zeros((B, v.words), dtype=torch.int32, device=dev),
                 logits=torch.zeros((B, v.n_tokens), dtype=torch.bfloat16, device=dev))
        lib.bind_state(d["states"], d["data"], d["length"], d["err"])
        return h, d

    def step(d):
        lib.advance_fill_argmax(d["tok"], d["mask"], d["logits"], d["tok"])

    def check(h, d, tokens, run):
        """One step from `tokens` (deep ones among them: private stacks that spill) through run()."""
        B = len(tokens)
        host = bf16_logits(rng, B, v.n_tokens)
        d["logits"].copy_(torch.from_numpy(host.view(np.int16)).to(dev).view(torch.bfloat16))
        d["tok"].copy_(torch.from_numpy(tokens))
        run()
        torch.cuda.synchronize()
        err = o.advance_batch(h["states"], h["data"], h["length"], tokens, v)
        mask = o.fill_mask(h["states"], h["data"], h["length"], v)
        assert (d["err"].cpu().numpy() == err).all() and (d["states"].cpu().numpy() == h["states"]).all()
        live = np.arange(cap)[None, :] < h["length"][:, None]
        assert (d["data"].cpu().numpy()[live] == h["data"][live]).all()
        assert (d["mask"].cpu().numpy().view(np.uint32) == mask).all()
        want = oracle_masked_argmax(host, mask, v.n_tokens)
        assert (d["tok"].cpu().numpy() == want).all()
        return want

    def some_tokens(B):
        return rng.choice([-1, *range(v.n_tokens - 7, v.n_tokens - 1), *rng.integers(0, v.n_tokens, 4)], size=B).astype(np.int32)

    big_h, big_d = batch(400)
    check(big_h, big_d, some_tokens(400), lambda: step(big_d))
    graph = torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(graph):
        step(big_d)
    small_h, small_d = batch(200)
    junk = [torch.full((1 << 18,), 0x7FFFFFFF, dtype=torch.int32, device=dev) for _ in range(16)]     # whoever takes freed memory
    for s in range(4):
        check(small_h, small_d, some_tokens(200), lambda: step(small_d))
        check(big_h, big_d, some_tokens(400), graph.replay)
    assert all(int((x != 0x7FFFFFFF).sum()) == 0 for x in junk)


@pytest.mark.gpu
def test_a_bind_that_fails_leaves_nothing_bound():
    """A batch whose workspaces exceed the device's memory is refused by the allocator; the calls on the handle then report
    that nothing is bound instead of running on the workspaces that the attempt released, and the next bind works."""
    import torch
    from paper_2506_03887_amd import Pre3, binding
    dev = torch.device("cuda:0")
    v, o, B, cap = _nesting_vocab(3000), Oracle(G.JSON), 6, 64
    lib = Pre3(G.JSON, v.bytes, v.offsets, v.eos_id, max_token_len=v.max_len, stack_cap=cap)
    s0 = lib.initial_state(0)
    s_d, err_d = torch.full((B,), s0, dtype=torch.int32, device=dev), torch.zeros(B, dtype=torch.int32, device=dev)
    d_d, l_d = torch.full((B, cap), s0, dtype=torch.int32, device=dev), torch.ones(B, dtype=torch.int32, device=dev)
    tok = torch.full((B,), v.tokens.index(b"[" * 17 + b"1"), dtype=torch.int32, device=dev)
    out, mask = torch.full_like(tok, -7), torch.zeros((B, v.words), dtype=torch.int32, device=dev)
    logits = torch.zeros((B, v.n_tokens), dtype=torch.bfloat16, device=dev)
    ids, jumped = torch.full((B, 4), -7, dtype=torch.int32, device=dev), torch.zeros((B, 8), dtype=torch.uint8, device=dev)
    lib.bind_state(s_d, d_d, l_d, err_d)
    too_many = 2 ** 31 - 1
    assert lib.workspace_bytes(too_many)["advance_spill"] > torch.cuda.get_device_properties(0).total_memory
    stacks = binding._Stacks(d_d.data_ptr(), l_d.data_ptr(), cap, too_many)       # the buffers are not read: no memory for the workspaces
    assert binding.load().pre3_bind_state(lib._h, s_d.data_ptr(), stacks, err_d.data_ptr()) == binding.E_HIP
    for call in (lambda: lib.advance(tok), lambda: lib.advance_fill_mask(tok, mask), lambda: lib.advance_fill_apply_mask(tok, mask, logits),
                 lambda: lib.advance_fill_argmax(tok, mask, logits, out), lambda: lib.apply_mask_argmax(logits, mask, out),
                 lambda: lib.apply_mask_topk(logits, mask, ids), lambda: lib.jump_forward(jumped, out), lambda: lib.step_is_one_kernel(logits)):
        with pytest.raises(binding.Pre3Error) as e:
            call()
        assert e.value.status == binding.E_BADARG
    torch.cuda.synchronize()
    assert int((out != -7).sum()) == 0 and int((s_d != s0).sum()) == 0 and int((l_d != 1).sum()) == 0
    lib.fill_apply_mask(s_d, d_d, l_d, mask, logits)                              # needs no binding
    want = o.fill_mask(np.full(B, s0, np.int32), np.full((B, cap), s0, np.int32), np.ones(B, np.int32), v)
    assert (mask.cpu().numpy().view(np.uint32) == want).all()
    lib.bind_state(s_d, d_d, l_d, err_d)
    lib.advance(tok)
    rc, stack = o.advance([s0], b"[" * 17 + b"1")
    assert rc == 0 and (l_d.cpu().numpy() == len(stack)).all() and int(err_d.abs().sum()) == 0
    assert (d_d[:, : len(stack)].cpu().numpy() == np.array(stack)[None, :]).all()


@pytest.mark.gpu
@pytest.mark.parametrize("V,options,expect", [
    # rows of 1, 3 and 5 blocks of 8,192 tokens; four blocks per compute unit are the limit of the spread form
    (8192, {}, {4: "spread", 256: "spread", 257: "spread", 1024: "spread", 1025: "two calls"}),
    (20_003, {}, {1: "spread", 63: "spread", 85: "spread", 86: "spread", 341: "spread", 342: "two calls"}),
    # ... three where the one kernel serves rows of at most 69,120 tokens
    (40_001, {}, {4: "spread", 63: "spread", 153: "spread", 154: "one kernel", 205: "one kernel", 256: "one kernel", 257: "two calls"}),
    (69_127, {}, {85: "spread", 86: "one kernel"}), (69_128, {}, {113: "spread", 114: "one kernel"}),
    (40_001, dict(row_threshold=64), {4: "two calls", 63: "two calls", 64: "one kernel", 256: "one kernel"}),       # id lists
    (40_001, dict(token_edges=False), {4: "two calls", 64: "two calls"})])
def test_the_query_names_the_kernel_that_runs(V, options, expect):
    """step_form against the names of the kernels that the two step calls launch, at both sides of every line of the rule;
    rows at 16-byte boundaries and rows one logit off them (which the one kernel does not serve)."""
    import torch
    from torch.profiler import ProfilerActivity, profile
    from paper_2506_03887_amd import Pre3
    dev = torch.device("cuda:0")
    assert torch.cuda.get_device_properties(0).multi_processor_count == 256
    v = _nesting_vocab(V)
    lib = Pre3(G.JSON, v.bytes, v.offsets, v.eos_id, max_token_len=v.max_len, stack_cap=16, **options)
    stride = -(-V // 8) * 8
    for B, form in expect.items():
        s0 = lib.initial_state(0)
        keep = (torch.full((B,), s0, dtype=torch.int32, device=dev), torch.full((B, 16), s0, dtype=torch.int32, device=dev),
                torch.ones(B, dtype=torch.int32, device=dev), torch.zeros(B, dtype=torch.int32, device=dev))
        lib.bind_state(*keep)
        mask = torch.zeros((B, v.words), dtype=torch.int32, device=dev)
        flat = torch.zeros(B * stride + 8, dtype=torch.int16, device=dev)
        tok = torch.full((B,), -1, dtype=torch.int32, device=dev)
        for off in (0, 1):
            logits = flat[off: off + B * stride].view(B, stride)
            for greedy in (False, True):
                want = form
                if form == "one kernel" and off == 1:
                    want = "spread" if B * -(-V // 8192) <= 1024 and not options else "two calls"
                # the greedy step takes the one kernel from half a row or more than one block per compute unit on, where that serves
                if greedy and form == "spread" and off == 0 and not options and 64 <= B <= 256 and (B >= 128 or B * -(-V // 8192) > 256):
                    want = "one kernel"
                assert lib.step_form(logits, greedy=greedy) == want, (B, off, greedy)
                run = (lambda: lib.advance_fill_argmax(tok, mask, logits, torch.empty_like(tok))) if greedy else \
                    (lambda: lib.advance_fill_apply_mask(tok, mask, logits))
                run()
                torch.cuda.synchronize()
                with profile(activities=[ProfilerActivity.CUDA]) as prof:
                    run()
                    torch.cuda.synchronize()
                names = " ".join(e.key for e in prof.key_averages())
                ran = "spread" if "step_spread_kernel" in names else "one kernel" if "advance_fill_apply_kernel" in names else "two calls"
                assert ran == want, (B, off, greedy, names)


def _bound(lib, B, cap):
    """Buffers of B sequences at their start, bound to lib: (states, length, data) and the mask and token buffers."""
    import torch
    dev = torch.device("cuda:0")
    states = torch.full((B,), lib.initial_state(0), dtype=torch.int32, device=dev)
    data = torch.zeros((B, cap), dtype=torch.int32, device=dev)
    data[:, 0] = states
    length, err = torch.ones(B, dtype=torch.int32, device=dev), torch.zeros(B, dtype=torch.int32, device=dev)
    lib.bind_state(states, data, length, err)
    return (states, length, data, err), torch.zeros((B, lib.words), dtype=torch.int32, device=dev), \
        torch.full((B,), -1, dtype=torch.int32, device=dev)


def _graph_us(call, n=8, rounds=5):
    """us per call, the fastest of a few replays of n calls in a graph."""
    import torch
    call()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        for _ in range(n):
            call()
    best = float("inf")
    for _ in range(rounds + 2):
        a, b = torch.cuda.Event(True), torch.cuda.Event(True)
        a.record()
        graph.replay()
        b.record()
        torch.cuda.synchronize()
        best = min(best, a.elapsed_time(b) * 1e3 / n)
    return best


@pytest.mark.gpu
def test_values_the_keys_cannot_decide_meet_across_the_blocks_of_a_row():
    """Zeros of either sign and NaN patterns on top of one block of a row (three blocks of 8,192 tokens), with equal, larger
    or no values in the others."""
    import torch
    from paper_2506_03887_amd import Pre3
    dev = torch.device("cuda:0")
    v, o, B = _nesting_vocab(20_003), Oracle(G.JSON), 16
    V = v.n_tokens
    lib = Pre3(G.JSON, v.bytes, v.offsets, v.eos_id, max_token_len=v.max_len, stack_cap=16)
    (states, length, data, _), mask_d, tok = _bound(lib, B, 16)
    mask = o.fill_mask(states.cpu().numpy(), data.cpu().numpy(), length.cpu().numpy(), v)
    ids = np.flatnonzero((mask[0][np.arange(V) >> 5] >> (np.arange(V) & 31).astype(np.uint32)) & 1)
    part = [ids[ids // 8192 == i] for i in range(3)]
    assert all(len(p) > 4 for p in part)
    host = np.full((B, V), 0xBF80, np.uint16)                                # -1
    host[0, part[1][2]], host[0, part[2][1]] = 0x8000, 0x0000                # -0 before +0
    host[1, part[1][2]], host[1, part[2][1]] = 0x0000, 0x8000                # +0 before -0
    host[2, part[0][3]], host[2, part[0][1]], host[2, part[1][0]] = 0x0000, 0x8000, 0x0000
    host[3, part[0]], host[3, part[1][3]] = 0x7FC1, 0x3F80                   # NaN around one value in another block
    host[4] = 0x7FC1                                                         # ... around -inf in the last
    host[4, part[2][2]] = 0xFF80
    host[5, part[0][0]], host[5, part[2][0]] = 0x0000, 0x3F80                # a zero beaten by another block
    host[6] = 0x7FC1                                                         # nothing but NaN
    host[7], host[7, part[2]] = 0xFF80, 0x8000                               # -inf, then zeros in the last block only
    host[8, part[1][1]], host[8, part[1][0]] = 0x7FC1, 0x0000
    host[9, part[2]] = np.where(np.arange(len(part[2])) % 2, 0x0000, 0x8000)
    host[10:] = bf16_logits(np.random.default_rng(3), B - 10, V)
    logits = torch.from_numpy(host.view(np.int16)).to(dev).view(torch.bfloat16)
    assert lib.step_form(logits, greedy=True) == "spread"
    for _ in range(2):                                                       # the counters are back at zero
        tok.fill_(-1)
        lib.advance_fill_argmax(tok, mask_d, logits, tok)
        assert (tok.cpu().numpy() == oracle_masked_argmax(host, mask, V)).all()


@pytest.mark.gpu
def test_a_zero_or_a_nan_on_top_costs_the_spread_greedy_step_little():
    """The block that holds such a value settles it on its own groups: 1.6 times the time of ordinary rows at 1 x 128,256
    (7 to 15 times when one block did that for the whole row).  The bound leaves room for a slow run."""
    import torch
    from paper_2506_03887_amd import Pre3
    v = _nesting_vocab(128_256)
    lib = Pre3(G.JSON, v.bytes, v.offsets, v.eos_id, max_token_len=v.max_len, stack_cap=16)
    us = {}
    for B in (1, 16):
        keep, mask, tok = _bound(lib, B, 16)
        logits = -torch.rand((B, v.n_tokens), dtype=torch.float32, device=tok.device).add_(0.5).to(torch.bfloat16)
        out = torch.empty_like(tok)
        assert lib.step_form(logits, greedy=True) == "spread"
        for kind, value in (("plain", 1.0), ("zero", 0.0), ("nan", float("nan"))):
            logits[:, ::7] = value
            us[kind] = _graph_us(lambda: lib.advance_fill_argmax(tok, mask, logits, out))
        assert max(us["zero"], us["nan"]) < 4 * us["plain"], (B, us)


@pytest.mark.gpu
def test_rows_left_open_are_walked_by_all_their_blocks():
    """Stacks for which the condition trees (cut at 3 entries) leave the whole vocabulary to the walk: every block of a row
    walks its own tokens, 0.07 times the time of the two calls (one wave per row) at 16 x 128,256; it was 1.02 when the
    last block did the row by itself.  The mask is the oracle's."""
    import torch
    from paper_2506_03887_amd import Pre3, apply_mask
    dev = torch.device("cuda:0")
    v, o, B, cap = _nesting_vocab(128_256), Oracle(G.JSON), 16, 64
    lib = Pre3(G.JSON, v.bytes, v.offsets, v.eos_id, max_token_len=v.max_len, stack_cap=cap, max_condition_depth=3)
    prefixes = [b'{"a":[1', b'[[{"b":"x', b'[[[12', b'{"k":{"l":[true', b'[{"q":[0', b'[[[["']
    stacks = [o.advance(o.initial_stack(0), prefixes[b % len(prefixes)])[1] for b in range(B)]
    left = [len(w) if ok else v.n_tokens for ok, _, w in (lib.debug_resolve_row(s) for s in stacks)]
    assert max(left) == v.n_tokens                                           # rows the tables have no answer for
    data = np.zeros((B, cap), np.int32)
    for b, s in enumerate(stacks):
        data[b, : len(s)] = s
    length = np.array([len(s) for s in stacks], np.int32)
    states = data[np.arange(B), length - 1].copy()
    s_d, d_d, l_d = (torch.from_numpy(x.copy()).to(dev) for x in (states, data, length))
    lib.bind_state(s_d, d_d, l_d, torch.zeros(B, dtype=torch.int32, device=dev))
    mask, tok = torch.zeros((B, v.words), dtype=torch.int32, device=dev), torch.full((B,), -1, dtype=torch.int32, device=dev)
    logits = torch.zeros((B, v.n_tokens), dtype=torch.bfloat16, device=dev)
    assert lib.step_form(logits) == "spread"

    def two_calls():
        lib.advance_fill_mask(tok, mask)
        apply_mask(logits, mask, v.n_tokens)

    spread = _graph_us(lambda: lib.advance_fill_apply_mask(tok, mask, logits), n=2, rounds=2)
    want = o.fill_mask(states, data, length, v)
    assert (mask.cpu().numpy().view(np.uint32) == want).all()
    assert spread < 0.5 * _graph_us(two_calls, n=2, rounds=2)


@pytest.mark.gpu
def test_a_refused_bind_keeps_the_earlier_binding():
    """Bad arguments leave what is bound as it is, an empty batch included."""
    import torch
    from paper_2506_03887_amd import Pre3, binding
    v, cap = _tiny_vocab(9), 16
    lib = Pre3(G.ARITHMETIC, v.bytes, v.offsets, v.eos_id, stack_cap=cap)
    (states, length, data, err), mask, tok = _bound(lib, 4, cap)
    bad = binding._Stacks(data.data_ptr(), length.data_ptr(), cap + 1, 4)                 # cap beyond stack_cap
    refuse = lambda: binding.load().pre3_bind_state(lib._h, states.data_ptr(), bad, err.data_ptr())
    tok.fill_(0)                                                                          # "a"
    assert refuse() == binding.E_BADARG
    lib.advance(tok)
    assert (length.cpu().numpy() == len(Oracle(G.ARITHMETIC).advance([lib.initial_state(0)], b"a")[1])).all()
    empty = torch.zeros((0, cap), dtype=torch.int32, device=tok.device)
    lib.bind_state(states[:0], empty, length[:0], err[:0])
    assert refuse() == binding.E_BADARG
    lib.advance(tok[:0])                                                                  # nothing to do, and no error
