"""Values that lanes of one wave hand over through LDS without a workgroup
barrier: in the kernel sources every wave barrier stands between a release fence
(the stores before it) and an acquire fence (the other lanes' loads after it)."""
import os
import re

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1105_2904_amd", "csrc")


def test_wave_barriers_stand_between_both_fences():
    fence = r'__builtin_amdgcn_fence\(__ATOMIC_%s, "workgroup"\);\s*'
    whole = re.compile(fence % "RELEASE" + r"__builtin_amdgcn_wave_barrier\(\);\s*" + fence % "ACQUIRE")
    seen = 0
    for name in sorted(os.listdir(CSRC)):
        with open(os.path.join(CSRC, name)) as f:
            text = f.read()
        bare = text.count("__builtin_amdgcn_wave_barrier()")
        assert len(whole.findall(text)) == bare, name
        seen += bare
    assert seen > 0
