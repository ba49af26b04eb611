"""The fp32 split kernel's ring of two slots for K and two for V in LDS: between a read of a slot by one wavefront and a write to it by
another, or the other way round, lies a workgroup barrier.  The wavefronts run freely between two barriers, so no run shows a missing one
reliably; here the order of reads, writes and barriers is taken from the kernel's source and every pair is looked at."""
import re

STAGES = 6


def _kernel(repo_root):
    text = open(f"{repo_root}/paper_2508_17756_amd/csrc/attention_f32_split.hip").read()
    text = re.sub(r"//[^\n]*", "", text)
    start, loop, end = text.index("next_offsets(0);"), text.index("for (int j = 0; j < n_blocks"), text.index("if (narrow) {")
    assert start < loop < end
    return text[start:loop], text[loop:end]


def _steps(part):
    """What a part of the kernel does to the ring, in the order of the source."""
    return re.findall(r"\b(stage_step|qk_product|pv_product|meet)\s*\(", part)


def _events(repo_root):
    """(read | write, slot) and barriers of the first STAGES iterations.  Staging with index j writes K of stage j + 2 and V of stage j + 1;
    QK of iteration j reads K of stage j + 1, PV V of stage j; stage s lies in slot s % 2.  The part in front of the loop stages with -2 (no V)
    and -1, and takes QK of stage 0."""
    prologue, loop = _kernel(repo_root)
    assert _steps(prologue)[0] == "stage_step" and _steps(prologue).count("stage_step") == 1
    events = []
    for step in _steps(prologue):
        if step == "stage_step":
            events += [("write", ("K", 0)), ("write", ("K", 1)), ("write", ("V", 0))]
        elif step == "qk_product":
            events.append(("read", ("K", 0)))
        else:
            assert step == "meet"
            events.append(step)
    for j in range(STAGES):
        for step in _steps(loop):
            if step == "stage_step":
                events += [("write", ("K", j % 2)), ("write", ("V", (j + 1) % 2))]
            elif step == "qk_product":
                events.append(("read", ("K", (j + 1) % 2)))
            elif step == "pv_product":
                events.append(("read", ("V", j % 2)))
            else:
                events.append(step)
    return events


def test_the_source_has_the_steps(repo_root):
    prologue, loop = _kernel(repo_root)
    assert sorted(set(_steps(loop))) == ["meet", "pv_product", "qk_product", "stage_step"]
    assert "(j & 1) * kStageBytes" in open(f"{repo_root}/paper_2508_17756_amd/csrc/attention_f32_split.hip").read()


def test_a_barrier_lies_between_reads_and_writes_of_a_slot(repo_root):
    since = []   # accesses since the last barrier
    for event in _events(repo_root):
        if event == "meet":
            since = []
            continue
        kind, slot = event
        for other, where in since:
            assert where != slot or other == kind, "%s of %s beside its %s" % (kind, slot, other)
        since.append(event)
