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
