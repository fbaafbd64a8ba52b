"""The library's unmangled symbols are the functions of include/mg.h: a helper
exported beside them could be replaced by another object's symbol of its name."""

import subprocess

import paper_1406_5369_amd as mg


def test_unmangled_exports_are_the_c_interface():
    out = subprocess.run(["nm", "-D", "--defined-only", mg.LIB_PATH], capture_output=True, text=True, check=True).stdout
    names = {line.split()[-1] for line in out.splitlines() if line.split()}
    # C++ names are mangled (_Z...); the compiler names each HIP object's code __hip_...
    plain = sorted(n for n in names if not n.startswith(("_Z", "__hip_")))
    assert plain == mg.header_functions()
