"""The hash that says whether a committed profile is of the present kernels."""
import os
import re
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2103_01691_amd", "csrc")


def test_hash_covers_every_kernel_a_profile_names():
    sys.path.insert(0, ROOT)
    import bench
    texts = {f: open(os.path.join(CSRC, f)).read() for f in os.listdir(CSRC) if f.endswith((".hip", ".inl", ".h"))}
    covered = {os.path.basename(s) for s in bench.KERNEL_SOURCES}
    named = set()
    for f in sorted(os.listdir(os.path.join(ROOT, "profiles"))):
        if f.endswith(".md"):
            named |= set(re.findall(r"\b\w+_kernel\b", open(os.path.join(ROOT, "profiles", f)).read()))
    ours = {k: [f for f, t in texts.items() if re.search(rf"void {k}\(", t)] for k in named}
    assert sum(1 for files in ours.values() if files) >= 4, ours
    for kernel, files in ours.items():
        # the file that defines it, those it includes and those that include it
        near = set(files)
        for _ in range(3):
            near |= {g for f in near for g in re.findall(r'#include "([^"]+)"', texts[f])}
            near |= {f for f, t in texts.items() if any(f'#include "{g}"' in t for g in near if g.endswith((".inl", ".h"))
                                                        and g != "mm_internal.h")}
        assert near <= covered, (kernel, sorted(near - covered))
