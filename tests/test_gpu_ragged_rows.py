"""GPU kernels on rows of logits that start at any 2-byte offset: vocabularies of odd size without padding,
views into larger buffers, sizes on both sides of a group (8), a line (64) and a block's span (2,048)."""
import numpy as np
import pytest

from oracle import apply_mask as oracle_apply_mask
from workloads.vocab import bf16_logits

pytestmark = pytest.mark.gpu


def _torch():
    import torch
    return torch, torch.device("cuda:0")


@pytest.mark.parametrize("V", [1, 7, 8, 9, 63, 64, 65, 2047, 2048, 2049, 6151])
@pytest.mark.parametrize("pad,offset", [(0, 0), (1, 0), (2, 1), (8, 0), (64, 64), (5, 61)])
def test_masked_rows_at_every_offset(V, pad, offset):
    """70 rows (with an odd stride their starts cover every offset within a 128-byte line), sparse, dense, empty and
    full masks: exactly the masked logits of each row change, and nothing around the rows."""
    torch, dev = _torch()
    from paper_2506_03887_amd import apply_mask
    rng = np.random.default_rng(V * 1000 + pad * 10 + offset)
    B, W, stride = 70, (V + 31) // 32, V + pad
    host = np.full((B, stride), 0x1234, dtype=np.uint16)
    host[:, :V] = bf16_logits(rng, B, V)
    mask = rng.integers(0, 2 ** 32, size=(B, W), dtype=np.uint64).astype(np.uint32)
    mask[::5] |= rng.integers(0, 2 ** 32, size=(14, W), dtype=np.uint64).astype(np.uint32) | np.uint32(0xFFFF)
    mask[1::5], mask[2::10] = 0, 0xFFFFFFFF
    flat = torch.full((B * stride + offset + 80,), 0x2345, dtype=torch.int16, device=dev)
    view = flat[offset: offset + B * stride].view(B, stride)
    view.copy_(torch.from_numpy(host.view(np.int16)).to(dev))
    apply_mask(view, torch.from_numpy(mask.view(np.int32)).to(dev), V)
    want = host.copy()
    oracle_apply_mask(want, mask, V)
    assert (view.cpu().numpy().view(np.uint16) == want).all()
    assert (flat[:offset] == 0x2345).all() and (flat[offset + B * stride:] == 0x2345).all()


@pytest.mark.parametrize("B", [65_528, 65_529, 131_100])
@pytest.mark.parametrize("V,stride", [(9, 9), (64, 64)])
def test_masked_rows_of_very_large_batches(B, V, stride):
    """More rows than one grid's second dimension holds go as several launches (rows at any offset, rows on 128-byte lines)."""
    torch, dev = _torch()
    from paper_2506_03887_amd import apply_mask
    rng = np.random.default_rng(B + V)
    host = bf16_logits(rng, B, stride)
    mask = rng.integers(0, 2 ** 32, size=(B, (V + 31) // 32), dtype=np.uint64).astype(np.uint32)
    rows = torch.from_numpy(host.view(np.int16)).to(dev)
    apply_mask(rows, torch.from_numpy(mask.view(np.int32)).to(dev), V)
    oracle_apply_mask(host, mask, V)
    assert (rows.cpu().numpy().view(np.uint16) == host).all()


@pytest.mark.parametrize("V,B", [(65, 3), (1003, 70), (40_005, 9), (20_011, 256), (131_071, 257)])
@pytest.mark.parametrize("pad,offset", [(0, 1), (3, 0), (16, 5)])
def test_sampled_rows_at_every_offset(V, B, pad, offset):
    """The greedy choice and the k best of rows that start off a 16-byte boundary: rows split over blocks, one block
    per row, and the row kept in registers (257 rows), special rows among them."""
    from test_gpu_argmax import _bound_lib, _special_logits, _special_masks
    from oracle import masked_argmax, masked_topk
    from workloads.vocab import Vocab
    torch, dev = _torch()
    rng = np.random.default_rng(V + B + pad)
    lib = _bound_lib(Vocab([bytes([97 + i % 5]) for i in range(V - 1)] + [b""], V - 1), B)
    stride = V + pad
    host = np.zeros((B, stride), dtype=np.uint16)
    host[:, :V] = bf16_logits(rng, B, V)
    W = (V + 31) // 32
    mask = rng.integers(0, 2 ** 32, size=(B, W), dtype=np.uint64).astype(np.uint32)
    head = min(B, 16)
    special, special_mask = _special_logits(rng, 16, V), _special_masks(rng, 16, V)
    host[:head, :V], mask[:head] = special[:head], special_mask[:head]
    mask[:, -1] &= np.uint32(0xFFFFFFFF >> (W * 32 - V))
    flat = torch.zeros(B * stride + offset + 16, dtype=torch.int16, device=dev)
    view = flat[offset: offset + B * stride].view(B, stride)
    view.copy_(torch.from_numpy(host.view(np.int16)).to(dev))
    logits, mask_d = view.view(torch.bfloat16), torch.from_numpy(mask.view(np.int32)).to(dev)
    tok = torch.empty(B, dtype=torch.int32, device=dev)
    lib.apply_mask_argmax(logits, mask_d, tok)
    assert tok.cpu().numpy().tolist() == masked_argmax(host, mask, V).tolist()
    for k in (1, 33, 64):
        ids, vals = torch.empty((B, k), dtype=torch.int32, device=dev), torch.empty((B, k), dtype=torch.int16, device=dev)
        lib.apply_mask_topk(logits, mask_d, ids, vals)
        want_ids, want_vals = masked_topk(host, mask, V, k)
        assert (ids.cpu().numpy() == want_ids).all() and (vals.cpu().numpy().view(np.uint16) == want_vals).all(), k


@pytest.mark.parametrize("V,B", [(7, 20), (8, 256), (9, 256), (15, 256), (64, 256), (8191, 256), (8192, 256), (8205, 256),
                                 (16_384, 17), (16_385, 17), (65_535, 256), (65_536, 17), (65_537, 17), (98_305, 17),
                                 (131_072, 256), (131_073, 17), (131_079, 48), (147_460, 17), (196_608, 48), (196_611, 48)])
def test_topk_of_rows_kept_in_registers(V, B):
    """A block per row (from four rows on up to 163,840 tokens), or several: rows with values of one sign only, few allowed tokens, hundreds of ties (the lists
    of the kernel run full), zeros of both signs, infinities, allowed NaN of both signs, and nothing allowed."""
    from test_gpu_argmax import _bound_lib
    from oracle import masked_topk
    from workloads.vocab import Vocab
    torch, dev = _torch()
    rng = np.random.default_rng(V)
    W = (V + 31) // 32
    lib = _bound_lib(Vocab([bytes([97 + i % 5]) for i in range(V - 1)] + [b""], V - 1), B)
    host = bf16_logits(rng, B, V)
    mask = rng.integers(0, 2 ** 32, size=(B, W), dtype=np.uint64).astype(np.uint32)
    host[1::16] |= 0x8000                                                   # below zero only
    host[2::16] = rng.choice([0x3F80, 0xBF80, 0x0000, 0x8000], size=host[2::16].shape)
    host[3::16, ::3] = 0x7FC1                                               # NaN of both signs, -inf, +inf
    host[3::16, 1::7] = 0xFFC1
    host[4::16, ::2] = 0xFF80
    host[5::16, 1::9] = 0x7F80
    host[6::16] = 0x3F80                                                    # one value everywhere
    for step, rows in ((2, slice(7, None, 16)), (8, slice(8, None, 16)), (12, slice(9, None, 16))):
        for _ in range(step):                                               # 1 in 4, in 256, in 4,096 of the tokens
            mask[rows] &= rng.integers(0, 2 ** 32, size=mask[rows].shape, dtype=np.uint64).astype(np.uint32)
    mask[10::16], mask[11::16] = 0, 0xFFFFFFFF
    mask[12::16] = 0
    mask[12::16, 0] = 0x00000101                                            # first tokens and the last
    mask[12::16, -1] |= np.uint32(1 << ((V - 1) & 31))
    mask[13::16] = 0
    mask[13::16, : max(1, W // 100)] = 0xFFFFFFFF                           # one run of ids
    host[14::16, : V // 2] |= 0x8000
    mask[:, -1] &= np.uint32(0xFFFFFFFF >> (W * 32 - V))
    logits, mask_d = torch.from_numpy(host.view(np.int16)).to(dev).view(torch.bfloat16), torch.from_numpy(mask.view(np.int32)).to(dev)
    for k in (1, 17, 64):
        if -(-V // 16384) * k > 1024:
            continue
        ids, vals = torch.empty((B, k), dtype=torch.int32, device=dev), torch.empty((B, k), dtype=torch.int16, device=dev)
        lib.apply_mask_topk(logits, mask_d, ids, vals)
        want_ids, want_vals = masked_topk(host, mask, V, k)
        bad = np.argwhere((ids.cpu().numpy() != want_ids) | (vals.cpu().numpy().view(np.uint16) != want_vals))
        assert len(bad) == 0, (k, bad[:4].tolist())


@pytest.mark.parametrize("V,B", [(131_080, 300), (147_457, 4), (163_839, 40), (163_840, 4), (163_841, 17), (163_848, 48), (262_147, 33),
                                  (131_080, 29), (163_840, 26), (163_840, 300)])
def test_topk_of_rows_at_the_longest_variant(V, B):
    """One block of twenty groups per row (aligned rows of more than 131,072 tokens whose narrow blocks would pass the compute units),
    or several blocks."""
    test_topk_of_rows_kept_in_registers(V, B)


@pytest.mark.parametrize("V,B,options", [(16_385, 9, {}), (33_033, 70, {}), (33_033, 600, {}), (65_569, 40, dict(max_condition_depth=2)),
                                         (100_003, 24, {}), (20_003, 30, dict(row_threshold=64))])
def test_mask_rows_off_a_16_byte_boundary(V, B, options):
    """pre3_fill_mask where rows of the bitmask start off a 16-byte boundary: rows in segments that are copied a word at a
    time, whole rows, rows with tokens or everything left open, id lists, finished and empty stacks."""
    from oracle import Oracle
    from paper_2506_03887_amd import Pre3
    from workloads import grammars as G
    from workloads.vocab import BASE_SEED, bpe_like_vocab
    torch, dev = _torch()
    v, o = bpe_like_vocab(V, 16, BASE_SEED + V), Oracle(G.JSON)
    assert v.words % 4 != 0
    lib = Pre3(G.JSON, v.bytes, v.offsets, v.eos_id, max_token_len=v.max_len, **options)
    prefixes = [b"", b"[", b'{"a":[1,', b'"abc', b"[[[[[[[[[[[[", b'{"a":{"b":"', b"12", b'[{"k":true},']
    data, length = np.zeros((B, 128), np.int32), np.ones(B, np.int32)
    for b in range(B):
        p = prefixes[b % len(prefixes)]
        st = o.advance(o.initial_stack(0), p)[1] if p else o.initial_stack(0)
        data[b, : len(st)], length[b] = st, len(st)
    states = data[np.arange(B), length - 1].copy()
    states[3::17] = -1                                                       # finished
    length[5::19] = 0                                                        # no stack
    m = torch.full((B + 1, v.words), 0x77777777, dtype=torch.int32, device=dev)
    s_d, d_d, l_d = (torch.from_numpy(x).to(dev) for x in (states, data, length))
    lib.fill_mask(s_d, d_d, l_d, m[:B])
    live = length > 0
    got, want = m.cpu().numpy().view(np.uint32), o.fill_mask(states[live], data[live], length[live], v)
    assert (got[:B][live] == want).all() and (got[:B][~live & (states >= 0)] == 0).all() and (got[B] == 0x77777777).all()
    assert lib.fault_count() == 0
