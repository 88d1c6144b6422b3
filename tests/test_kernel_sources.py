"""Rules of the kernel sources that no run can show reliably."""
import os
import re

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2512_09904_amd", "csrc")


def kernels():
    """Name and body of every __global__ function."""
    out = {}
    for f in sorted(os.listdir(CSRC)):
        if not f.endswith(".hip"):
            continue
        src = re.sub(r"//[^\n]*", "", open(os.path.join(CSRC, f)).read())
        for m in re.finditer(r"__global__[^;{]*?\b(k_\w+)\s*\([^{]*\{", src):
            depth, end = 1, m.end()
            while depth:
                depth += {"{": 1, "}": -1}.get(src[end], 0)
                end += 1
            out[m.group(1)] = src[m.end():end]
    return out


def test_kernels_that_raise_flags_decide_once_per_workgroup():
    """Whether a solve is still live is read from its flags.  In a launch that
    itself raises flags two wavefronts of a workgroup may read them differently;
    where the wavefronts take indices from each other through LDS, the ones that
    stay would follow what the others never wrote.  Such kernels take one
    decision per workgroup (live_block); the others that raise flags share
    nothing but the sums of a solve that has faulted."""
    ks = kernels()
    raising = {k for k, b in ks.items() if "raise_flag(" in b}
    sums_only = {"k_pose", "k_fold", "k_end"}
    assert {"k_build", "k_visc_heat", "k_momentum"} <= raising
    for k in sorted(raising - sums_only):
        own = re.findall(r"\b(SLOT_PROLOGUE|live|live_sub)\s*\(", ks[k])
        assert not own and "live_block(" in ks[k], f"{k}: a wavefront decides for itself ({own})"
