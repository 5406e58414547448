"""Where an LM head finishes its logits in the GEMM, and where it takes partial sums: host code, no GPU needed.  256 compute units."""
import ctypes as C
import os

import pytest

import paper_2408_08146_amd as K


@pytest.fixture(autouse=True)
def _built():
    if not os.path.exists(K.library_path()):
        from paper_2408_08146_amd.build import build_library
        build_library(verbose=False)


def groups(vocab, hidden, rows, sequences=8):
    """candidates of a row from the joined form, 0: partial sums"""
    return C.CDLL(K.library_path()).kt_head_groups(vocab, hidden, rows, sequences * hidden // 128, 256)


@pytest.mark.parametrize("hidden", [512, 1024, 2048, 4096, 6656])
def test_large_vocabularies_are_joined(hidden):
    for rows in (1, 17, 33, 64, 66, 132, 240, 480, 512):
        for vocab in (20000, 24000, 32000):
            joined = groups(vocab, hidden, rows)
            assert joined or (hidden >= 4096 and rows >= 66 and vocab < 32000)   # in three splits there
            assert joined <= 1024


def test_many_rows_of_few_workgroups_take_partial_sums():
    """Measured with one layer: 240 rows, 4096 columns, 8000 tokens 212 us against 236 joined in three splits; 512 rows 292 and
    325 in two; 132 rows, 512 columns, 1000 tokens 77 and 79 in twelve whole workgroups"""
    for vocab, hidden, rows in ((8000, 4096, 240), (16000, 4096, 240), (8000, 4096, 512), (8000, 6656, 512), (1000, 512, 132), (1000, 1024, 66),
                                (4000, 512, 66), (4000, 2048, 512)):
        assert groups(vocab, hidden, rows) == 0
    for vocab, hidden, rows in ((4000, 512, 240), (4000, 512, 480), (8000, 1024, 132), (12000, 2048, 240), (12000, 512, 66)):
        assert groups(vocab, hidden, rows) > 0


def test_a_row_tile_of_64_by_columns_and_workgroups():
    """33 to 64 rows, measured: 4000 tokens 77 us against 72 joined at 2048 columns, 104 and 106 at 4096"""
    for rows in (33, 48, 64):
        assert groups(4000, 512, rows) and groups(4000, 2048, rows) and groups(2000, 2048, rows) and groups(8000, 4096, rows)
        assert not groups(4000, 4096, rows) and not groups(4000, 6656, rows) and not groups(8000, 6656, rows)
        assert groups(12000, 6656, rows)
        assert not groups(50000, 512, rows)   # more than a round of workgroups
    for rows in (1, 16, 32):
        assert groups(2000, 6656, rows)
