"""What launches ask of the runtime beside the launch itself (no GPU): a kernel's grant of LDS is one for all its calls, whichever
thread makes them."""
from launches import Grant, Launch, traced
from paper_2511_06345_amd import inputs as gen


def test_a_call_does_not_lower_what_another_was_granted():
    steps = [step for call in traced([("conv1d", gen.BF16, 31, 17, 1862, 39, Kw, 1, 0, 1) for Kw in (7, 6, 7)]) for step in call]
    launches = [step for step in steps if isinstance(step, Launch) and step.lds > 65536]
    assert len(launches) == 3 and len({step.kernel for step in launches}) == 1, steps
    assert launches[0].lds > launches[1].lds, "the calls are meant to differ in what they take"
    granted = [step for step in steps if isinstance(step, Grant)]
    # before the kernel's first launch, and not again
    assert granted == [Grant(launches[0].kernel, granted[0].bytes)] and granted[0].bytes >= launches[0].lds, granted
    assert steps.index(granted[0]) < steps.index(launches[0])
