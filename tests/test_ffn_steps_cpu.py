"""The order in which the grouped FFN's scheduling waves look a unit up, checked on the host for every length of the contraction."""
import os
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2508_17624_amd", "csrc")
STEPS = ("claim", "entry", "rows", "stored", "publish")             # as the kernels run them inside a slab
MOST = 520


@pytest.fixture(scope="module")
def places(tmp_path_factory):
    """{kernel: {slabs: the slab of each step}} from the header that the kernels include."""
    cxx = shutil.which("g++") or shutil.which("c++")
    if not cxx:
        pytest.skip("no host compiler")
    d = tmp_path_factory.mktemp("steps")
    src, exe = d / "steps.cpp", d / "steps"
    src.write_text('#include "ffn_steps.h"\n#include <cstdio>\nint main() {\n  for (int nk = 2; nk <= %d; ++nk) {\n'
                   "    const ew::SchedSteps s[2] = {ew::steps_spread(nk), ew::steps_late(nk)};\n"
                   '    for (int i = 0; i < 2; ++i) std::printf("%%d %%d %%d %%d %%d %%d %%d\\n", i, nk, s[i].claim, s[i].entry, s[i].rows, s[i].stored, s[i].publish);\n'
                   "  }\n}\n" % MOST)
    subprocess.run([cxx, "-std=c++17", "-I", CSRC, str(src), "-o", str(exe)], check=True, timeout=60)
    out = {"k_ffn_dec": {}, "k_ffn_big": {}}
    for line in subprocess.run([str(exe)], check=True, capture_output=True, text=True, timeout=60).stdout.splitlines():
        i, nk, *at = map(int, line.split())
        out[list(out)[i]][nk] = dict(zip(STEPS, at))
    return out


@pytest.mark.parametrize("kernel", ["k_ffn_dec", "k_ffn_big"])
def test_a_unit_is_published_with_what_was_looked_up_for_it(places, kernel):
    """Three units of nk slabs one after the other: every publication happens in the last slab but one, once per unit, and its entry,
    rows and completion counter belong to the unit claimed last, not to the one claimed before."""
    assert sorted(places[kernel]) == list(range(2, MOST + 1))
    for nk, at in places[kernel].items():
        known = dict.fromkeys(STEPS[:-1], 0)                          # the unit that each result is of
        published = []
        for unit in (1, 2, 3):
            for kt in range(nk):
                for i, step in enumerate(STEPS):
                    if at[step] != kt:
                        continue
                    if step == "claim":
                        known["claim"] = unit
                    elif step == "publish":
                        assert kt == nk - 2 and set(known.values()) == {unit}, f"{nk} slabs, unit {unit}: {known}"
                        published.append(unit)
                    else:
                        known[step] = known[STEPS[i - 1]]
        assert published == [1, 2, 3], f"{nk} slabs"
