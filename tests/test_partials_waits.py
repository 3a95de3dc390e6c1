"""Between a share's partial stores and the count that publishes them every thread has to wait for its
stores: a workgroup barrier alone does not (its release is of workgroup scope).  Read off the assembly
of the kernels built here."""
import re

from tests.test_kernel_resources import compiled_kernels


def test_partial_stores_are_waited_for_before_they_are_counted():
    assert waited_counts("attention_mfma.hip") >= 5      # four decode builds and the wide kernel


def test_kernels_that_hand_partials_to_a_second_launch_keep_no_counters():
    """Counters outlive a call: one left in a bad state by another kernel's time-out would leave rows unwritten."""
    text, kernels = compiled_kernels("attention_split.hip")
    assert sum("pv_attn_mfma" in name for name in kernels) == 4
    assert "atomic" not in "\n".join(ln.split(";")[0] for ln in text.split("\n"))


def waited_counts(source):
    text, kernels = compiled_kernels(source)
    lines = text.split("\n")
    checked = 0
    for name in kernels:
        if "pv_attn_mfma" not in name:
            continue
        start = next(i for i, ln in enumerate(lines) if ln.startswith(name + ":"))
        end = next(i for i in range(start, len(lines)) if lines[i].startswith(".Lfunc_end"))
        body = [ln.split(";")[0].strip() for ln in lines[start:end]]
        for i, ln in enumerate(body):
            # every count that follows write-through (sc1) stores without another barrier in between
            if "global_atomic_add" not in ln:
                continue
            barrier = max(j for j in range(i) if body[j] == "s_barrier")
            stores = [j for j in range(barrier) if re.match(r"(buffer|global)_store_\w+ .*\bsc1\b", body[j])]
            if not stores or any(body[j] == "s_barrier" for j in range(stores[-1], barrier)):
                continue
            assert any("s_waitcnt vmcnt(0)" in body[j] for j in range(stores[-1], barrier)), (name, i)
            checked += 1
    return checked
