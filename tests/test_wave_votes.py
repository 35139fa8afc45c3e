"""The kernels' wave-wide operations are asked of all lanes: none stands behind a condition that lanes decide one by one."""
import glob
import os
import re

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
WIDE = re.compile(r"\b(?:__ballot|__any|__all|__shfl\w*|wave_scan|wave_sum|last_lane|lane_value|dpp_or_zero|"
                  r"__builtin_amdgcn_read(?:first)?lane|__builtin_amdgcn_update_dpp|__syncthreads\w*)\b[^;(]*\(")


def behind_a_condition(text):
    """Statements with such an operation to the right of &&, || or ?, unless template constants alone stand to the left."""
    text = re.sub(r"//[^\n]*", "", text)
    found = []
    for m in WIDE.finditer(text):
        before = re.split(r"[;{}]", text[:m.start()])[-1]
        guard = re.search(r"(.*)(?:&&|\|\||\?)", before, re.S)
        if guard and not re.fullmatch(r"[\s(!&|]*(?:(?:if|while)\s*\()?[\s(!&|]*[A-Z_]+[\s)]*", guard.group(1)):
            found.append(" ".join((before + m.group(0)).split()))
    return found


def test_a_vote_behind_a_lane_s_condition_is_seen():
    """`lane == 0 && __ballot(mine) == 0` asks lane 0 alone, and two lanes then wrote the same three words of LDS."""
    assert behind_a_condition("x = 1; if (mine || (lane == 0 && __ballot(mine) == 0)) { s = 1; }")
    assert behind_a_condition("const uint32_t n = lane < 4 ? wave_sum(c) : 0u;")
    assert not behind_a_condition("if (!RK && __ballot(kmax >= 7u) && lane == 0) a();")
    assert not behind_a_condition("n = wave_sum(lane < 4 ? c : 0u);")


def test_votes_of_the_kernels():
    sources = glob.glob(os.path.join(ROOT, "paper_2402_11857_amd", "csrc", "**", "*.h*"), recursive=True)
    assert len(sources) > 5
    for path in sources:
        with open(path) as f:
            assert behind_a_condition(f.read()) == [], os.path.basename(path)
