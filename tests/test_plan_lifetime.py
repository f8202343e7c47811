"""What a plan asks of the HIP runtime between its creation and its end (no GPU: see launch_recorder)."""
import pytest

import launch_recorder as rec

DISABLE_SYSTEM_FENCE = 0x20000000     # hipEventDisableSystemFence


@pytest.fixture(scope="module")
def stand_in(tmp_path_factory):
    return rec.build_stand_in(tmp_path_factory.mktemp("recorder"))


@pytest.mark.parametrize("block", [False, True])
def test_a_refill_waits_for_an_event_that_orders_memory(stand_in, block):
    """The copy that overwrites a list is ordered behind the launches that read it, and behind the draw counters that they wrote, by
    the event alone: an event without its fence is documented to time work, not to synchronise with it."""
    program = """
pack = lambda n: ([n] * 8, [n] * 8, [n] * 8, [0] * 8) if args[0] else ([n] * 8,)
plan = BlockPlan(*pack(900), 8, 8, 128) if args[0] else Plan(*pack(900), 8, 8, 128)
plan.forward(); plan.backward()
for n in (900, 700, 800, 600, 900, 500):
    plan.update(*pack(n)); plan.forward(); plan.backward()
out(calls())
"""
    calls = rec.record(stand_in, program, block)[0]
    events = [n for what, _, n in calls if what == "event"]
    assert len(events) == 3 and not any(n & DISABLE_SYSTEM_FENCE for n in events), [hex(n) for n in events]
    # three slots: from the fourth list on, a copy comes behind the wait for its slot's last launch
    order = "".join({"copy": "c", "wait": "w", "launch": "l", "mark": "m"}.get(what, "") for what, _, _ in calls)
    assert order.count("c") == 7 and order.count("w") == 4, order
    assert order.replace("l", "").replace("m", "") == "ccc" + "wc" * 4, order


@pytest.mark.parametrize("lengths", [[17, 64, 111], [900] * 8, [0]])
def test_destroying_a_plan_waits_for_the_device(stand_in, lengths):
    """As the header says, also where the lists never were on the device: a caller may free the tensors of its launches next."""
    program = """
plan = Plan(args[0], 8, 8, 128)
plan.forward()
calls()
plan.destroy()
out([what for what, _, _ in calls()])
"""
    calls = rec.record(stand_in, program, lengths)[0]
    assert "free" in calls or "sync" in calls, calls
