"""Counts of items that a level's value product deals a group's chunks of eight members to, read from the workspace size (one fp32 output
per item): they follow what was measured per count (us, whole / in 2 / 4 / 8)."""
import pytest

import paper_2506_21411_amd as dchag


def splits(monkeypatch, B, C, N, D, heads, g):
    need = lambda: dchag.dchag_workspace_bytes(dchag.DCHAG_BF16, B, C, N, 1, 1, D, heads, [g], 0)
    monkeypatch.delenv("DCHAG_VAGG_SPLIT", raising=False)
    total = need()
    monkeypatch.setenv("DCHAG_VAGG_SPLIT", "1")
    whole = need()
    monkeypatch.delenv("DCHAG_VAGG_SPLIT")
    part = B * -(-C // g) * N * D * 4
    assert (total - whole) % part == 0
    return max(1, (total - whole) // part), total


@pytest.mark.parametrize("shape,count", [
    ((4, 64, 256, 1024, 16, 32), 1),      # 256 items of 4 chunks: 154 / 160 / 164
    ((2, 96, 200, 1024, 16, 24), 1),      # 224 of 3: 115 / 137
    ((3, 80, 128, 2048, 16, 40), 1),      # 192 of 5 (two would take three chunks, and six in all): 281 / 326 / 336
    ((1, 256, 300, 1024, 16, 128), 8),    # 80 of 16: 402 / 275 / 287 / 255
    ((1, 256, 300, 2048, 16, 128), 4),    # 160 of 16: 797 / 851 / 722
    ((2, 64, 256, 256, 8, 64), 8),        # 16 of 8, the shortest chunks: 95 / 78 / 68 / 64
    ((1, 512, 256, 256, 8, 64), 4),       # 64 of 8: 106 / 91 / 83 / 86
    ((1, 256, 256, 256, 8, 16), 1),       # 128 of 2: 42.4 / 43.6
    ((1, 9, 32, 256, 8, 9), 2),           # fewer chunks than counts
])
def test_count_by_measured_cost(shape, count, monkeypatch):
    assert splits(monkeypatch, *shape)[0] == count


def test_static_scratch_is_not_outgrown(monkeypatch):
    """80 items of 64 chunks, whose softmax weights take 21 MB: eight would leave the 32 MB of dchag_aggregate_level_static, two stay inside."""
    count, total = splits(monkeypatch, 1, 1024, 300, 1024, 16, 512)
    assert count == 2 and total <= dchag.STATIC_SCRATCH_BYTES
