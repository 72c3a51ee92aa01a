"""Plans of lists that no sample starts (more than 32 keys), through the workspace they
ask for (no GPU): such lists cost each chunk a start from nothing, so their chunks are
only short where the chip would be idle, and 17 or more FP16 reads of a tile take 128
of them at most."""
import pytest

from paper_2603_22245_amd import _lib as L

from test_score_workspace import _index

KEYS, SMALL = 64 * 8, 512  # bytes of a list, and of everything else per read (260)


@pytest.mark.parametrize("k_fetch", [33, 64])
@pytest.mark.parametrize("precision,n_windows,n_reads,chunks", [
    ("fp16", 200_000, 32, 128), ("fp16", 200_000, 60, 128), ("fp16", 10_000_000, 100, 128),
    ("fp16", 200_000, 8_000, 17), ("fp16", 42_000, 8_000, 17), ("fp8", 42_000, 8_000, 17),
    ("fp8", 1_000_000, 8_000, 17), ("fp32", 200_000, 8_000, 17), ("fp16", 200_000, 3_000, 44)])
def test_chunks_of_cold_lists(precision, k_fetch, n_windows, n_reads, chunks):
    idx = _index(precision, n_windows)
    assert L.rm_score_workspace_bytes(idx, n_reads, k_fetch) <= n_reads * (chunks * KEYS + SMALL) + 1024
