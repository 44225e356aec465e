"""The launch an LSTM layer's recurrence gets on the CUs of a stream's mask (host only): the workgroups of the one
launch wait for each other, so they must all fit the CUs at once."""
import pytest

import paper_2304_13541_amd as ds


def slots(*js, byte=0xff):
    return sum(byte << (8 * j) for j in js)


def test_masks_with_a_part_of_a_slot_go_step_by_step():
    """4 CUs in each of 32 slots are 128 CUs, not the 256 that the count of slots says; nor is a mask of whole slots
    and a part of one counted."""
    for byte in (0x0f, 0x01, 0x7f, 0xfe):
        cus = 32 * bin(byte).count("1")
        assert ds.lstm_plan(50, 32, 1024, cus, slots(*range(32), byte=byte)) == (0, 0)
    assert ds.lstm_plan(50, 4, 256, 60, slots(*range(7)) | slots(7, byte=0x0f)) == (0, 0)


@pytest.mark.parametrize("n", range(1, 33))
def test_whole_slots(n):
    """Consecutive slots: as planned from their number; the workgroups fit one to a CU of the engines that hold the
    fewest (slot j on engine j % 4)."""
    for T, B, H in [(50, 32, 1024), (50, 16, 1024), (4, 1, 32), (9, 17, 96), (20, 5, 2048), (7, 32, 512)]:
        got = ds.lstm_plan(T, B, H, 8 * n, slots(*range(n)))
        assert got == ds.lstm_plan(T, B, H, 8 * n)
        room = 8 * (n if n < 4 else n // 4 * 4)
        rt, blocks = got
        groups, ksw = (B + 15) // 16, (H + 255) // 256
        allowed = [r for r in (2, 4, 8) if (r == 2 or ksw <= 4) and groups * (H // 4 // r) <= room]
        assert (rt, blocks) == ((allowed[0], groups * (H // 4 // allowed[0])) if allowed else (0, 0))


def test_scattered_slots():
    """Two slots of one engine and one of another hold 16 workgroups, not 24; short sequences go step by step."""
    assert ds.lstm_plan(6, 4, 128, 24, slots(0, 1, 4)) == (2, 16)
    assert ds.lstm_plan(6, 4, 160, 24, slots(0, 1, 4)) == (4, 10)
    assert ds.lstm_plan(3, 4, 128, 24, slots(0, 1, 4)) == (0, 0)
    for bad in ((0, 1, 32), (4, 0, 32), (4, 33, 32), (4, 1, 48), (4, 1, 4096)):
        with pytest.raises(ds.DStackError):
            ds.lstm_plan(*bad)
