"""The build's list of files: every local header that a source reaches is in it, so that a change of any of
them changes the hash that keys the autotuner's on-disk cache."""
import os
import re

from paper_2204_14241_amd import build


def test_every_included_header_is_hashed():
    todo, seen = list(build.SOURCES), set()
    while todo:
        f = os.path.normpath(todo.pop())
        if f in seen:
            continue
        seen.add(f)
        with open(f) as fh:
            for inc in re.findall(r'^\s*#include\s+"([^"]+)"', fh.read(), re.M):
                found = [p for p in (os.path.join(os.path.dirname(f), inc), os.path.join(build.ROOT, "include", inc))
                         if os.path.exists(p)]
                assert found, (f, inc)
                todo.append(found[0])
    listed = {os.path.normpath(f) for f in build.DEPS}
    assert seen <= listed, seen - listed
    assert len(build.DEPS) == len(listed)
