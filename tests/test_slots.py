"""The slots that the runs of a process share (rewl_slots.h, built for the host)."""


def test_slots_are_bounded_and_used_again(kernel_arith):
    assert kernel_arith.slots_in_order() == 0


def test_slots_are_never_held_twice(kernel_arith):
    assert kernel_arith.slots_shared(8, 3000) == 0
