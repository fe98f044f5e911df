"""The walk over the parts of a list of rays (csrc/ltm_parts.h): every group is taken once
and in order, no part is tried twice, and past a bad group the parts grow again."""
import os
import subprocess

import pytest

import paper_1812_03358_amd as pkg

CSRC = os.path.join(os.path.dirname(pkg.__file__), "csrc")
# argv: the number of groups, then the bad ones; a line "begin end ok" for each part
MAIN = r"""
#include "ltm_parts.h"
#include <cstdio>
#include <cstdlib>
int main(int argc, char** argv)
{
    for (Parts p{std::atoi(argv[1])}; !p.done();) {
        bool ok = true;
        for (int i = 2; i < argc; ++i)
            ok = ok && !(std::atoi(argv[i]) >= p.begin() && std::atoi(argv[i]) < p.end());
        const bool halve = !ok && p.end() - p.begin() > 1;
        std::printf("%d %d %d\n", p.begin(), p.end(), halve ? 0 : 1);
        halve ? p.halve() : p.next();
    }
}
"""


@pytest.fixture(scope="module")
def walk(tmp_path_factory):
    d = tmp_path_factory.mktemp("parts")
    (d / "main.cpp").write_text(MAIN)
    subprocess.run(["g++", "-std=c++17", "-I", CSRC, "-o", str(d / "main"), str(d / "main.cpp")], check=True)

    def run(groups, bad):
        out = subprocess.run([str(d / "main"), str(groups), *map(str, bad)], check=True,
                             capture_output=True, text=True, timeout=10).stdout
        return [tuple(map(int, line.split())) for line in out.splitlines()]
    return run


@pytest.mark.parametrize("groups", [1, 2, 3, 5, 25, 32, 33, 143, 144])
def test_walk(walk, groups):
    depth = (groups - 1).bit_length()
    for bad in ([], [0], [groups - 1], [groups // 2], [0, groups // 3], list(range(groups))):
        tried = walk(groups, bad)
        assert len({t[:2] for t in tried}) == len(tried)
        at = 0
        for b, e, ok in tried:
            assert b == at and e > b
            at = e if ok else at
        assert at == groups
        # a whole list in one part; a bad group at each level: the part with it and the
        # one beside it
        assert len(tried) <= 1 + 2 * depth * len(set(bad))
