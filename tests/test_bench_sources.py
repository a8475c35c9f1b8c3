"""The benchmark's recorded counters are valid for the kernels they were taken
on: every source that makes or picks a standalone-solve kernel is in its hash."""
import os

import bench
from paper_2609_15217_amd import build


def test_hash_covers_the_kernels_and_their_choice(tmp_path):
    names = ("thread_", "lanes_", "narrow_")
    units = [s for s in build.generate(str(tmp_path)) if os.path.basename(s).startswith(names)]
    need = {os.path.relpath(h, build.ROOT) for u in units for h in build._local_headers(u)}
    # the files of the dispatch rules: where a choice among kernels is made
    for f in sorted(os.listdir(build.CSRC)):
        if "Choice auto_choice(" in open(os.path.join(build.CSRC, f)).read():
            need.add(os.path.relpath(os.path.join(build.CSRC, f), build.ROOT))
    missing = need - set(bench.KERNEL_SOURCES)
    assert not missing, missing
    for rel in bench.KERNEL_SOURCES:
        assert os.path.exists(os.path.join(build.ROOT, rel)), rel
