"""The build's and the benchmark's lists of source files: every file the library is compiled from is
in the build's, so that an edit rebuilds it, and every file the walks are made of is in the benchmark's,
whose hash decides whether committed counters still describe them."""
from __future__ import annotations

import os
import re

import bench
from paper_2604_13929_amd import build

CSRC = build.CSRC


def _includes(path):
    """The files of csrc and include that a source names, with theirs."""
    seen, todo = set(), [path]
    while todo:
        f = todo.pop()
        with open(f) as fh:
            for name in re.findall(r'^\s*#include "([^"]+)"', fh.read(), re.M):
                for d in (CSRC, build.INCLUDE):
                    p = os.path.join(d, name)
                    if os.path.exists(p) and p not in seen:
                        seen.add(p)
                        todo.append(p)
    return seen


def test_build_lists_every_source():
    sources = {os.path.join(CSRC, f) for f in os.listdir(CSRC) if f.endswith(".hip")}
    assert set(build.SOURCES) == sources
    headers = set().union(*(_includes(s) for s in sources))
    assert set(build.HEADERS) == headers
    assert headers >= {os.path.join(CSRC, f) for f in os.listdir(CSRC) if f.endswith(".hpp")}


def test_bench_hashes_every_file_of_the_walks():
    walks = [os.path.join(CSRC, f) for f in ("photonmc.hip", "batch.hip", "cells.hip")]
    files = set(walks).union(*(_includes(s) for s in walks)) - {os.path.join(build.INCLUDE, "spinodal.h")}
    assert {os.path.join(bench.ROOT, f) for f in bench.SOURCES} == files
