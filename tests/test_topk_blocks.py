"""The blocks that rows of logits are cut into for the k best: the rule's lines (host code, no GPU), and on the GPU every
form of a long row against the oracle on rows at and off 16-byte boundaries."""
import ctypes

import pytest


def _groups(V, batch, aligned):
    from paper_2506_03887_amd import load
    rule = load()["_ZN4pre318masked_topk_groupsEiibi"]
    rule.restype, rule.argtypes = ctypes.c_int, [ctypes.c_int, ctypes.c_int, ctypes.c_bool, ctypes.c_int]
    return rule(V, batch, aligned, 256)


@pytest.mark.parametrize("V,batch,aligned,groups", [
    (1, 1, True, 4), (16_384, 300, False, 4), (16_385, 1, False, 8), (65_537, 1, True, 12), (98_305, 256, False, 16), (131_072, 256, False, 16),
    # small batches of the rows that one block streams longest: narrow blocks that hand over
    (114_688, 1, True, 16), (114_689, 16, True, 4), (114_689, 17, False, 16), (131_072, 16, False, 4), (131_072, 17, True, 16), (131_073, 1, True, 4),
    (131_073, 28, True, 4), (131_073, 29, True, 20), (147_456, 28, False, 4), (147_457, 25, True, 4), (147_457, 26, True, 20), (152_064, 24, True, 4),
    # one block of twenty groups: aligned rows
    (143_360, 40, True, 20), (163_840, 25, True, 4), (163_840, 26, True, 20), (163_840, 512, True, 20),
    # other rows: segments, two blocks a row, and twenty groups where two blocks a row do not fit the chip at once
    (131_073, 1, False, 4), (160_003, 31, False, 4), (131_075, 32, False, 12), (160_003, 128, False, 12), (160_003, 129, False, 20),
    (163_840, 256, False, 20), (163_840, 512, False, 20),
    # longer rows
    (163_841, 31, True, 4), (163_841, 300, True, 12), (196_609, 300, True, 16), (262_144, 300, False, 16), (262_145, 64, True, 16),
    (262_145, 85, True, 16), (262_145, 86, True, 20), (280_000, 128, False, 20), (280_000, 256, True, 20), (400_000, 100, True, 16), (500_000, 64, True, 16)])
def test_lines_of_the_rule(V, batch, aligned, groups):
    assert _groups(V, batch, aligned) == groups


def test_which_rows_are_merged_by_a_launch_of_their_own():
    from paper_2506_03887_amd import load
    rule = load()["_ZN4pre324masked_topk_merged_apartEiii"]
    rule.restype, rule.argtypes = ctypes.c_bool, [ctypes.c_int] * 3
    assert not rule(256, 2, 256) and rule(257, 2, 256) and not rule(31, 16, 256) and rule(31, 17, 256) and not rule(1, 62, 256)


@pytest.mark.gpu
@pytest.mark.parametrize("V,B,pad,offset", [(163_849, 256, 0, 0), (163_849, 257, 7, 0), (400_000, 31, 0, 0), (500_003, 130, 0, 1),
                                            (143_360, 3, 0, 0), (163_840, 3, 8, 0), (143_363, 5, 0, 1), (163_839, 33, 0, 0), (131_073, 129, 0, 3),
                                            (262_149, 86, 3, 0), (262_149, 33, 0, 0)])
def test_rows_of_either_form(V, B, pad, offset):
    """Rows with ties at the bound, few allowed tokens, the best in the last group of a block or in the rest of the row."""
    import numpy as np
    import torch
    from oracle import masked_topk
    from test_gpu_argmax import _bound_lib
    from workloads.vocab import Vocab, bf16_logits
    dev, rng, W, stride = torch.device("cuda:0"), np.random.default_rng(V + B), (V + 31) // 32, V + pad
    lib = _bound_lib(Vocab([bytes([97 + i % 5]) for i in range(V - 1)] + [b""], V - 1), B)
    host = bf16_logits(rng, B, stride)
    mask = rng.integers(0, 2 ** 32, size=(B, W), dtype=np.uint64).astype(np.uint32)
    edges = [t for e in (16_384, 98_304, 131_072, 163_840) for t in (e - 8, e - 1, e, e + 7) if t < V] + [V - V % 8 - 1, V - 1]
    host[:, rng.choice(edges, size=6, replace=False)] = 0x4300
    host[1::8] = rng.choice([0x3F80, 0xBF80, 0x0000, 0x8000], size=host[1::8].shape)
    host[2::8] |= 0x8000
    mask[3::8] &= rng.integers(0, 2 ** 32, size=mask[3::8].shape, dtype=np.uint64).astype(np.uint32)
    mask[4::8] = 0
    mask[4::8, [0, W - 1]] = 0xFFFF
    mask[:, -1] &= np.uint32(0xFFFFFFFF >> (W * 32 - V))
    flat = torch.zeros(B * stride + offset, dtype=torch.int16, device=dev)
    view = flat[offset:].view(B, stride)
    view.copy_(torch.from_numpy(host.view(np.int16)).to(dev))
    mask_d = torch.from_numpy(mask.view(np.int32)).to(dev)
    for k in (1, min(50, 1024 // -(-V // 16_384))):
        ids, vals = torch.empty((B, k), dtype=torch.int32, device=dev), torch.empty((B, k), dtype=torch.int16, device=dev)
        lib.apply_mask_topk(view.view(torch.bfloat16), mask_d, ids, vals)
        want_ids, want_vals = masked_topk(host, mask, V, k)
        assert (ids.cpu().numpy() == want_ids).all() and (vals.cpu().numpy().view(np.uint16) == want_vals).all(), k
