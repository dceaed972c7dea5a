"""Counts that the lanes of one wave hand to each other through LDS, with no workgroup barrier between: every
such store and the loads before and after it stand on their own sides of wave_lds_order(), which is what keeps
the compiler from moving one across (the language orders no thread's load against another thread's store).
Checked in the source, as a compiled kernel only shows what one compiler made of it."""

import os
import re

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_front_end_ranks_are_ordered_between_steps():
    src = open(os.path.join(ROOT, "paper_2608_24938_amd", "csrc", "k_route.hip")).read()
    body = src[src.index("void decode_front_kernel("):]
    step = body[body.index("int rank[STEPS];"):]
    step = step[: step.index("lds_barrier();")]                # the loop over the wave's slots
    events = re.findall(r"=\s*wcnt\[wave\]\[te\]|wcnt\[wave\]\[te\]\s*=|wave_lds_order\(\)", step)
    kinds = ["order" if e.startswith("wave") else "load" if e.startswith("=") else "store" for e in events]
    assert kinds == ["load", "order", "store", "order"], kinds


def test_wave_lds_order_fences_both_sides():
    src = open(os.path.join(ROOT, "paper_2608_24938_amd", "csrc", "common.hpp")).read()
    body = src[src.index("void wave_lds_order() {"):]
    body = body[: body.index("}\n")]
    assert re.findall(r"fence\(__ATOMIC_(\w+), \"wavefront\", \"local\"\)|(wave_barrier)", body) == [
        ("RELEASE", ""), ("", "wave_barrier"), ("ACQUIRE", "")]
