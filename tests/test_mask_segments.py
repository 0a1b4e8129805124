"""How many blocks make a row of pre3_fill_mask: half of the grid's blocks serve tables that determine every token, all of
them tables with leaves that leave more than 64 tokens to the walk (one wave walks a segment's tokens).  Host code, no GPU."""
import ctypes

import pytest

from workloads import grammars as G
from workloads.vocab import BASE_SEED, bpe_like_vocab

UNITS = 256                                # compute units of a host-only handle


def _segments(lib, batch):
    from paper_2506_03887_amd import load
    rule = load()["_ZN4pre322fill_mask_row_segmentsEPK11pre3_handlei"]
    rule.restype, rule.argtypes = ctypes.c_int, [ctypes.c_void_p, ctypes.c_int]
    return rule(lib._h, batch)


def _most(V, batch, blocks):
    """The most segments of at least 8,192 tokens with which `batch` rows (in eights) come to no more than `blocks`."""
    vec = -(-(-(-V // 32)) // 4)
    n = max(1, min(blocks // (-(-batch // 8) * 8), -(-vec // 64)))
    return -(-vec // -(-vec // n))


@pytest.mark.parametrize("options,opens", [({}, False), (dict(max_condition_depth=3), True), (dict(max_condition_depth=8), True),
                                           (dict(max_condition_depth=30), False), (dict(row_threshold=64), False)])
@pytest.mark.parametrize("V", [20_003, 66_001])
def test_rows_that_may_be_walked_keep_all_blocks(V, options, opens):
    from paper_2506_03887_amd import Pre3
    v = bpe_like_vocab(V, 16, BASE_SEED + V)
    lib = Pre3(G.JSON, v.bytes, v.offsets, v.eos_id, max_token_len=v.max_len, host_only=True, **options)
    blocks = 4 * UNITS if opens else 2 * UNITS
    for batch in (1, 8, 40, 66, 96, 128, 130, 200, 256, 257, 264, 320, 341, 342, 500, 512, 513, 1024, 2000):
        assert _segments(lib, batch) == _most(V, batch, blocks), batch
    assert _segments(lib, 320) == (3 if opens else 1)
