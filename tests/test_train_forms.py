"""Which of its two kernels a training product takes, and in how many K splits: host code, no GPU needed."""
import ctypes as C

import pytest

import paper_2408_08146_amd as K


def form(rows, cols, terms, strided=False, room=1 << 30):
    """(row tiles of a workgroup, 0 where the product is not streamed; splits), as the library's own rule gives them"""
    f = C.CDLL(K.library_path()).kt_product_form
    f.argtypes, f.restype = [C.c_int] * 4 + [C.c_size_t, C.POINTER(C.c_int)], C.c_int
    splits = C.c_int()
    tiles = f(rows, cols, terms, int(strided), room, C.byref(splits))
    return tiles, splits.value


@pytest.fixture(autouse=True)
def _built():
    import os
    if not os.path.exists(K.library_path()):
        from paper_2408_08146_amd.build import build_library
        build_library(verbose=False)


def test_few_stages_over_few_columns_are_not_streamed():
    """One split over 4000 columns of 512 terms, the logits of a small head: 20.1 us for the forward pass against 22.3
    streamed."""
    for rows in (1, 4, 10, 20, 32):
        assert form(rows, 4000, 512, room=0) == (0, 1)
        assert form(rows, 300, 64, room=0) == (0, 1)


def test_large_products_are_streamed():
    for rows in (1, 20, 64, 128, 300):
        assert form(rows, 32000, 4096, room=0) == (min(8, max(2, -(-rows // 16))), 1)
        assert form(rows, 1024, 32000)[0]
        assert form(rows, 4096, 32000, strided=True)[0]


def test_splits_go_by_the_die_with_the_most_workgroups():
    """The 12 column tiles of 1500 columns lie on eight dies, two on some: sixteen splits fill those, more make a second round
    there.  The product of 128 rows took 106 us in 24 splits and 85 in 16."""
    streamed, splits = form(128, 1500, 32000)
    assert streamed and splits == 16
    streamed, splits = form(128, 4000, 32000)   # 32 tiles, four a die
    assert streamed and splits == 8


@pytest.mark.parametrize("strided", [False, True])
def test_every_split_has_work_and_room(strided):
    """Over the sizes that the training calls take: splits fit their room, leave each at least two chunks of 32 (streamed:
    two stages of 64), and what the streaming kernel cannot take stays away from it."""
    sizes = (1, 2, 31, 32, 33, 63, 64, 65, 127, 128, 300, 1000, 4001, 12345, 32000)
    for rows in (1, 16, 17, 32, 33, 64, 65, 128, 129, 300, 600):
        for cols in sizes:
            for terms in sizes:
                for room in (0, 2 * rows * cols, 1 << 34):
                    streamed, splits = form(rows, cols, terms, strided, room)
                    assert 1 <= splits <= 32
                    if splits > 1:
                        assert splits * rows * cols <= room
                        assert -(-terms // (64 if streamed else 32)) >= 2 * splits
                    if streamed:
                        assert cols >= 32 and terms >= 64
    assert not form(20, 1 << 23, 64, strided)[0] and not form(20, 64, 1 << 23, strided)[0]
