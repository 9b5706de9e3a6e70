"""The kernels' machine code as the compiler leaves it (compiled here, no GPU).

The compiler keeps a vector operation two wait states away from the compare
that writes the lane mask it reads, but it does not look into inline assembly:
code written there has to keep that distance itself, or the operation can see
an older mask."""
import os
import re
import subprocess

import pytest

from paper_2409_03771_amd import build as B

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
pytestmark = pytest.mark.skipif(not os.path.exists(HIPCC), reason="no hipcc")


@pytest.fixture(scope="module", params=["cc.hip", "segment.hip"])
def code(request, tmp_path_factory):
    out = tmp_path_factory.mktemp("asm") / "out.s"
    flags = [f for f in B.FLAGS if f not in ("-fPIC", "-shared")]
    subprocess.check_call([HIPCC, *flags, "-S", "--cuda-device-only", "-o",
                           str(out), os.path.join(B.CSRC, request.param)])
    return request.param, out.read_text().splitlines()


WAIT_STATES = 2


def mask_hazards(lines):
    """Vector operations that read a lane mask fewer than WAIT_STATES wait
    states after the compare that wrote it: (line number, text)."""
    found, recent = [], {}
    for no, line in enumerate(lines, 1):
        text = line.split(";")[0].strip()
        if not text or text.startswith("."):
            continue
        if text.endswith(":"):  # a label: what comes before is another path
            recent = {}
            continue
        op, _, rest = text.partition(" ")
        op = op.strip()
        args = [a.strip() for a in rest.split(",")]
        if op.startswith("v_"):
            carries = re.match(r"v_(mad_[ui]64|div_scale|\w+_co_)", op)
            reads = args[2 if carries else 1:]  # (a carry out comes second)
            if op.startswith("v_cndmask") and op.endswith("_e32"):
                reads = reads + ["vcc"]
            for a in reads:
                if recent.get(a, WAIT_STATES) < WAIT_STATES:
                    found.append((no, text))
        step = int(args[0], 0) + 1 if op == "s_nop" else 1
        recent = {m: n + step for m, n in recent.items()
                  if n + step < WAIT_STATES}
        if op.startswith("v_cmp_"):
            recent[args[0]] = 0
    return found


def test_the_check_itself():
    near = ["v_cmp_lt_f32_e64 s[2:3], v1, v2",
            "v_addc_co_u32 v0, vcc, v0, v0, s[2:3]"]
    assert len(mask_hazards(near)) == 1
    assert len(mask_hazards([near[0], "s_nop 0", near[1]])) == 1
    assert mask_hazards([near[0],
                         "v_mad_u64_u32 v[4:5], s[2:3], v3, s12, v[2:3]"]) == []
    assert mask_hazards([near[0], "s_nop 1", near[1]]) == []
    assert mask_hazards([near[0], "v_mov_b32 v4, v5", "s_mov_b32 s9, 0",
                         near[1]]) == []
    assert len(mask_hazards(["v_cmp_eq_u32_e32 vcc, 0, v1",
                             "v_cndmask_b32_e32 v2, v3, v4, vcc"])) >= 1


def test_masks_are_read_two_wait_states_after_the_compare(code):
    name, lines = code
    assert sum(bool(re.match(r"\s*v_cmp_", s)) for s in lines) > 50, name
    bad = mask_hazards(lines)
    assert not bad, f"{name}: {len(bad)}, e.g. {bad[:3]}"


def test_link_tables_are_aligned_for_their_wide_loads(code):
    name, lines = code
    if name != "cc.hip":
        pytest.skip("the tables are in cc.hip")
    at = next(i for i, s in enumerate(lines)
              if re.match(r"_ZN\S*kLink\S*:", s))
    align = next(s for s in reversed(lines[:at]) if ".p2align" in s)
    assert int(re.search(r"\.p2align\s+(\d+)", align).group(1)) >= 4, align
