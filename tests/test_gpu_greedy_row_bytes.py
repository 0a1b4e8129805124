"""The greedy step with one row to a unit, whose waves go on by themselves when the plan is there and mask what they hold with the
materialised row's bytes (ten to seventeen groups of logits per lane; shorter rows meet first): lockstep with the oracle at the edges
of the variants' rows, the best token alone, twice in a lane, in
two lanes, in two waves and beside masked tokens of the same value, and on rows that are put together in LDS after all (id lists,
open rows, finished sequences, all in one batch)."""
import numpy as np
import pytest

from oracle import Oracle, masked_argmax as oracle_masked_argmax
from test_gpu_greedy_two_rows import _vocab
from workloads import grammars as G
from workloads.vocab import bf16_logits

pytestmark = pytest.mark.gpu

LANES = 960


@pytest.mark.parametrize("V,B,pad,offset,options", [
    (8 * 8 * LANES + 8, 256, 0, 0, {}), (8 * 9 * LANES + 7, 129, 1, 0, {}), (8 * 9 * LANES + 8, 130, 0, 0, dict(compact_cycles=True)),
    (8 * 16 * LANES + 5, 200, 3, 0, {}), (8 * 17 * LANES + 7, 66, 1, 0, {}), (8 * 17 * LANES + 8, 90, 0, 0, {}), (100_003, 97, 0, 3, {}),
    (70_000, 128, 0, 0, dict(row_threshold=64)), (70_003, 128, 5, 0, dict(max_condition_depth=3))])
def test_greedy_step_on_materialised_and_other_rows(V, B, pad, offset, options):
    import torch
    from paper_2506_03887_amd import Pre3
    dev, cap = torch.device("cuda:0"), 48
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
    assert lib.step_form(view, greedy=True) == "one kernel"
    tokens = np.full(B, -1, np.int32)
    for s in range(5):
        err = o.advance_batch(states, data, length, tokens, v)
        mask = o.fill_mask(states, data, length, v)
        host = bf16_logits(rng, B, stride)
        for b in range(B):
            allowed = np.flatnonzero((mask[b, np.arange(V) >> 5] >> (np.arange(V) & 31).astype(np.uint32)) & 1)
            if len(allowed) == 0 or b % 8 == 0:
                continue
            t = int(allowed[-1] if b % 8 == 1 else allowed[0] if b % 8 == 2 else rng.choice(allowed))
            group, k = divmod(t, 8)
            same = {3: [group * 8 + (k + 1) % 8, group * 8 + (k + 3) % 8],                     # its own group, masked ones among them
                    4: [(group + LANES) * 8 + k, (group + 2 * LANES) * 8 + k],                 # the same lane's later groups
                    5: [(group + 1) * 8, (group + 63) * 8 + 7], 6: [(group + 64) * 8, (group + 5 * 64) * 8 + 1],   # other lanes, other waves
                    7: list(rng.choice(V, size=2000))}.get(b % 8, [])
            host[b, [x for x in [t, *same] if x < V]] = 0x4300 if s % 2 else 0xBF80 if b % 8 == 7 else 0x42C0
            if s % 2 == 0 and b % 8 == 7:
                host[b] |= 0x8000
        view.copy_(torch.from_numpy(host.view(np.int16)).to(dev).view(torch.bfloat16))
        lib.advance_fill_argmax(tok_d, mask_d, view, tok_d)
        want, got = oracle_masked_argmax(host, mask, V), tok_d.cpu().numpy()
        assert (got == want).all(), (s, np.flatnonzero(got != want)[:5], got[got != want][:5], want[got != want][:5])
        assert (err_d.cpu().numpy() == err).all() and (s_d.cpu().numpy() == states).all() and (l_d.cpu().numpy() == length).all(), s
        live = np.arange(cap)[None, :] < length[:, None]
        assert (d_d.cpu().numpy()[live] == data[live]).all() and (mask_d.cpu().numpy().view(np.uint32) == mask).all(), s
        tokens = want.copy()
        tokens[rng.random(B) < 0.15] = v.eos_id         # some end (and stay finished), some are refused it
        tok_d.copy_(torch.from_numpy(tokens))
    assert lib.fault_count() == 0


@pytest.mark.parametrize("V,B", [(70_000, 128), (128_256, 256)])
def test_equal_logits(V, B):
    """Rows of one value (the best token is the first allowed one, every lane holds the best), of a value that half of the allowed
    tokens have, of one that only the partial group and another lane's groups have, and of what the keys cannot decide: the oracle's
    tokens, and a step takes no more than twice as long as on random logits (with the lanes that hold the best looked at one after the
    other: nine times)."""
    import torch
    from paper_2506_03887_amd import Pre3
    dev, cap, V = torch.device("cuda:0"), 48, V + 3
    if torch.cuda.get_device_properties(0).multi_processor_count != 256:
        pytest.skip("the lines of the dispatch are drawn for 256 compute units")
    v, o = _vocab(V), Oracle(G.JSON)
    lib = Pre3(G.JSON, v.bytes, v.offsets, v.eos_id, max_token_len=v.max_len, stack_cap=cap)
    text = o.advance(o.initial_stack(0), b'["a')[1]          # inside a string: most tokens are allowed
    data = np.zeros((B, cap), np.int32)
    data[:, : len(text)] = text
    d_d, l_d = torch.from_numpy(data).to(dev), torch.full((B,), len(text), dtype=torch.int32, device=dev)
    s_d, err_d = d_d[:, len(text) - 1].contiguous(), torch.zeros(B, dtype=torch.int32, device=dev)
    lib.bind_state(s_d, d_d, l_d, err_d)
    mask_d, out_d = torch.zeros((B, v.words), dtype=torch.int32, device=dev), torch.zeros(B, dtype=torch.int32, device=dev)
    none = torch.full((B,), v.eos_id, dtype=torch.int32, device=dev)       # refused here: the stacks stay as they are
    mask = o.fill_mask(s_d.cpu().numpy(), data, np.full(B, len(text), np.int32), v)
    allowed = np.flatnonzero((mask[0, np.arange(V) >> 5] >> (np.arange(V) & 31).astype(np.uint32)) & 1)
    assert len(allowed) > V // 3
    rng = np.random.default_rng(V)
    logits = torch.zeros((B, V + 5), dtype=torch.bfloat16, device=dev)[:, :V]
    assert lib.step_form(logits, greedy=True) == "one kernel"

    def step():
        lib.advance_fill_argmax(none, mask_d, logits, out_d)

    def us_per_step():
        for _ in range(5):
            step()
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        times = []
        for _ in range(7):
            a.record()
            for _ in range(20):
                step()
            b.record()
            b.synchronize()
            times.append(a.elapsed_time(b) * 50)
        return sorted(times)[3]

    took = {}
    for kind in ("random", "equal", "half", "ends", "zeros", "nan"):
        host = bf16_logits(rng, B, V)
        if kind == "equal":
            host[:] = np.where(np.arange(B) % 2, 0x4000, 0xC000)[:, None]
        elif kind == "half":
            host[rng.random(host.shape) < 0.5] = 0x4300
        elif kind == "ends":
            host[:, np.append(allowed[-1:], allowed[-1:] - np.arange(1, 4) * 8 * LANES)] = 0x4300
        elif kind == "zeros":                               # the largest allowed value, either sign
            host |= 0x8000
            host[:, ::7], host[:, 3::7] = 0x0000, 0x8000
        elif kind == "nan":
            host[:, ::1000], host[:, 5::1000] = 0x7FC0, 0xFFC0
        logits.copy_(torch.from_numpy(host.view(np.int16)).to(dev).view(torch.bfloat16))
        step()
        assert (out_d.cpu().numpy() == oracle_masked_argmax(host, mask, V)).all(), kind
        assert (mask_d.cpu().numpy().view(np.uint32) == mask).all() and (err_d.cpu().numpy() == 1).all(), kind
        took[kind] = us_per_step()
    print(took)
    compared = took.pop("zeros"), took.pop("nan")               # rows that are gone through a second time, as numbers
    assert max(compared) < 8 * took["random"] and max(took.values()) < 2 * took["random"], took
