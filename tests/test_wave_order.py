"""Lanes of one wave that exchange values through LDS need a memory fence
beside the wave barrier: the barrier alone is no memory operation to the
compiler, which may then move a lane's load over another lane's store."""
import glob
import os
import re

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                    "paper_2207_07098_amd", "csrc")


def test_every_wave_barrier_is_fenced():
    found = 0
    for path in sorted(glob.glob(os.path.join(CSRC, "*"))):
        if not path.endswith((".hip", ".h", ".cpp")):
            continue
        with open(path) as f:
            code = re.sub(r"//[^\n]*", "", f.read())
        stmts = [q.strip() for q in code.replace("{", ";").split(";")]
        for q, s in enumerate(stmts):
            if "__builtin_amdgcn_wave_barrier" not in s:
                continue
            found += 1
            where = "%s: barrier %d" % (os.path.basename(path), found)
            assert stmts[q - 1] == '__builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront")', where
            assert stmts[q + 1] == '__builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront")', where
    assert found                       # the local solves exchange values this way
