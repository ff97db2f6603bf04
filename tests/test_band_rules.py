"""The rules by which pilc_twar_inverse decodes the bands of tall images (csrc/pilc_twar_rules.hpp), compiled with the host
compiler and held against the figures that stand beside them."""
import os
import re
import subprocess

import pytest

RULES = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2206_05279_amd", "csrc",
                     "pilc_twar_rules.hpp")

_PROGRAM = """
#include <cstdio>
#include "%s"
int main()
{
    unsigned strips, bands, columns;
    while (scanf("%%u %%u %%u", &strips, &bands, &columns) == 3) {
        const unsigned blocks = (columns + 63u + 15u) / 16u;
        const pilc::BandLaunch l = pilc::band_launches(strips, bands, blocks);
        const char *way = pilc::bands_one_at_a_time(strips, bands, blocks) ? "one"
                          : pilc::bands_alone_on_a_unit(l.strips, l.bands, blocks) ? "alone" : "two";
        printf("%%s %%llu %%u %%llu\\n", way, (unsigned long long)l.strips, l.bands, (unsigned long long)l.launches);
    }
}
""" % RULES


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    at = tmp_path_factory.mktemp("rules")
    (at / "rules.cpp").write_text(_PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-Wall", "-Werror", "-o", str(at / "rules"), str(at / "rules.cpp")], check=True)

    def ask(shapes):
        text = "".join("%d %d %d\n" % s for s in shapes)
        out = subprocess.run([str(at / "rules")], input=text, capture_output=True, text=True, check=True).stdout
        return [(a, int(b), int(c), int(d)) for a, b, c, d in (line.split() for line in out.splitlines())]
    return ask


def test_rules_take_what_was_measured_to_be_fast(rules):
    rows = re.findall(r"^//\s+(\d+) x\s+(\d+) x\s+(\d+)\s+(\d+)\s+(\d+)\s+(\d+)\s+(one|two|alone)$", open(RULES).read(), re.M)
    assert len(rows) >= 60
    for row, (way, _, _, _) in zip(rows, rules([tuple(map(int, r[:3])) for r in rows])):
        times = dict(zip(("one", "two", "alone"), map(int, row[3:6])))
        assert way == row[6], row
        assert times[way] <= 1.1 * min(times.values()), row


def test_launches_hold_their_words(rules):
    """Every launch of bands together has at least two bands, fits the words, and the launches have all strips."""
    shapes = [(s, b, w) for s in (1, 2, 63, 256, 400, 70000) for b in (2, 3, 17, 32, 300, 67108864) for w in (1, 16, 400, 2047, 65535)]
    words = int(re.search(r"kBandWords = 1u << (\d+)", open(RULES).read()).group(1))
    for (strips, bands, columns), (_, each, together, launches) in zip(shapes, rules(shapes)):
        assert 2 <= together <= bands and each * launches >= strips > each * (launches - 1)
        assert each * together * 16 * ((columns + 78) // 16) <= 1 << words


def test_lines_on_the_gpu_are_the_lines_of_the_rules(rules):
    """test_gpu_twar.py's shapes for either side of a line are on either side of one: each has a neighbour in the list, at one
    dimension, that goes another way."""
    text = open(os.path.join(os.path.dirname(os.path.abspath(__file__)), "test_gpu_twar.py")).read()
    shapes = [tuple(map(int, t)) for t in re.findall(r"\((\d+), (\d+), (\d+)\)", text[text.index("LINES = ["):text.index("LINES + [")])]
    assert len(shapes) >= 50
    ways = dict(zip(shapes, (r[0] for r in rules([(n, -(-h // 64), w) for n, h, w in shapes]))))
    for a in shapes:
        near = [b for b in shapes if b != a and sum(x != y for x, y in zip(a, b)) == 1
                and max(abs(x - y) for x, y in zip(a, b)) <= 2]
        assert any(ways[b] != ways[a] for b in near), (a, ways[a])
