"""The library's host-side choices (csrc/rules.hpp), compiled into a small
program: no GPU."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def run(tmp_path, body):
    src, exe = tmp_path / "rules.cpp", tmp_path / "rules"
    src.write_text('#include <cstdio>\n#include "%s/paper_2210_04892_amd/csrc/rules.hpp"\n'
                   "using namespace mlfma;\nint main() {\n%s\nreturn 0; }\n" % (ROOT, body))
    subprocess.run(["g++", "-std=c++17", "-Wall", "-Werror", str(src), "-o", str(exe)], check=True)
    return subprocess.run([str(exe)], check=True, capture_output=True, text=True).stdout.split("\n")[:-1]


# tiled kernel, or the group table: 0 sibling sets of 4, 2 merged groups of 8
TILED, SETS, MERGED = -1, 0, 2


@pytest.mark.parametrize("option", ["AUTO", "GROUPS", "LDS"])
@pytest.mark.parametrize("single", [True, False])
def test_translation_of_few_vectors(tmp_path, option, single):
    """A handle tuned to the LDS-operator shape: the tiled kernel takes one
    right-hand side (and two in single precision) only where the tuner was
    free to choose it."""
    sizes, counts = [100, 10000, 10001], [1, 2, 4, 5, 16]
    body = "TunedTrans t{8, 2, 2, 8, 1};\n"
    for boxes in sizes:
        for n in counts:
            body += ("{ auto s = trans_shape(MLFMA_TRANS_%s, t, %s, %d, %d, true);"
                     ' std::printf("%%d %%d\\n", s.gi, s.lds); }\n' % (option, str(single).lower(), boxes, n))
    got = [tuple(map(int, r.split())) for r in run(tmp_path, body)]
    want = []
    for boxes in sizes:
        for n in counts:
            if option == "AUTO" and (n == 1 or (n == 2 and single and boxes <= 10000)):
                want.append((TILED, 0))
            elif n < (2 if single else 5):
                want.append((SETS if boxes <= 10000 else MERGED, 0))
            else:
                want.append((MERGED, 1))
    assert got == want


def test_translation_of_other_shapes(tmp_path):
    """Tiled handles run the tiled kernel, except in lockstep batches, which
    share launches of the group kernel; register and matrix-core shapes stay."""
    body = 'auto p = [](TransShape s) { std::printf("%d %d %d %d\\n", s.gi, s.rb, s.rw, s.lds); };\n'
    for n in (1, 2, 16):
        body += "p(trans_shape(MLFMA_TRANS_TILED, TunedTrans{}, true, 100, %d, true));\n" % n
        body += "p(trans_shape(MLFMA_TRANS_AUTO, TunedTrans{}, true, 100, %d, false));\n" % n
        body += "p(trans_shape(MLFMA_TRANS_AUTO, TunedTrans{4, 0, 1, 2, 0}, true, 100, %d, true));\n" % n
        body += "p(trans_shape(MLFMA_TRANS_MATRIX, TunedTrans{16, 3, 4, 1, 0}, false, 100, %d, true));\n" % n
        body += "p(trans_shape(MLFMA_TRANS_AUTO, TunedTrans{8, 2, 2, 8, 1}, false, 100, %d, false));\n" % n
    got = run(tmp_path, body)
    for i, n in enumerate((1, 2, 16)):
        assert got[5 * i:5 * i + 5] == ["-1 1 0 0", "0 1 0 0", "0 1 2 0", "3 4 1 0", "2 2 8 1" if n == 16 else "0 1 0 0"]


def slots(tmp_path, state, padded, plain, io, budget):
    """(slot, grow, released slots) for slots [(busy, arena, io)]."""
    body = "std::vector<SlotSize> s{%s};\n" % ", ".join("{%d, %d, %d}" % c for c in state)
    body += "SlotPick p = pick_slot(s, %d, %d, %d, %d, %d);\n" % (
        padded, plain, io, sum(a + 2 * b for _, a, b in state), budget)
    body += 'std::printf("%d %d", p.slot, p.grow); for (int i : p.release) std::printf(" %d", i); std::printf("\\n");\n'
    out = [int(v) for v in run(tmp_path, body)[0].split()]
    return out[0], bool(out[1]), out[2:]


@pytest.mark.parametrize("state,want", [
    ([(0, 100, 10)], (0, False, [])),                            # an arena that could not be had padded is kept
    ([(0, 100, 10), (0, 106, 10)], (1, False, [])),              # padded rows where a slot has the room
    ([(1, 106, 10), (0, 100, 10)], (1, False, [])),              # a busy one is not waited for
    ([(0, 99, 10), (0, 0, 0)], (0, True, [])),                   # too small without padding either
    ([(0, 106, 9)], (0, True, [])),                              # buffers too small
    ([(1, 106, 10)], (-1, False, [])),
])
def test_slot_without_budget(tmp_path, state, want):
    assert slots(tmp_path, state, 106, 100, 10, 0) == want


@pytest.mark.parametrize("state,budget,want", [
    ([(0, 100, 10)], 120, (0, False, [])),
    ([(0, 60, 5), (0, 0, 0)], 200, (0, True, [])),
    ([(1, 60, 5), (0, 0, 0)], 190, (1, True, [])),               # 70 + 120
    ([(1, 60, 5), (0, 0, 0)], 189, (-1, False, [])),
    ([(1, 60, 5), (0, 20, 0), (0, 30, 0)], 190, (1, True, [2])),  # the other idle slot makes room
    ([(0, 0, 0)], 119, (-1, False, [])),
])
def test_slot_within_budget(tmp_path, state, budget, want):
    assert slots(tmp_path, state, 100, 100, 10, budget) == want


@pytest.mark.parametrize("memory,want", [
    (126, "106"),    # padded arena and both buffers
    (125, "100"),    # the padded arena fits, the buffers after it do not
    (105, "0"),
    (119, "0"),
])
def test_slot_buffers(tmp_path, memory, want):
    """Whatever is tried and given up is freed again."""
    body = """
long long left = %d;
std::vector<std::pair<char *, unsigned long long>> held;
char *next = nullptr;
auto alloc = [&](unsigned long long n) -> char * {
    if ((long long)n > left) return nullptr;
    left -= n;
    held.push_back({++next, n});
    return next;
};
auto release = [&](char *p) {
    for (auto &h : held) if (h.first == p) left += h.second, h.second = 0;
};
SlotBuffers b;
bool ok = alloc_slot(106, 100, 10, alloc, release, b);
std::printf("%%llu %%d %%lld\\n", b.arena_bytes, ok, left);
""" % memory
    got = run(tmp_path, body)[0].split()
    assert got == [want, str(int(want != "0")), str(memory - (int(want) + 20 if want != "0" else 0))]


@pytest.mark.parametrize("free,padding,want", [(100, 0, "1 0"), (95, 6, "1 6"), (95, 0, "0 0"), (90, 6, "0 6")])
def test_padding_given_up_for_memory(tmp_path, free, padding, want):
    """An allocation of 100: got, and padding given up."""
    body = """
int left = %d, padding = %d, given = 0;
void *p = alloc_or_unpad([&]() -> void * { return left >= 100 ? &left : nullptr; },
                         [&] { given = padding; left += padding; return padding > 0; });
std::printf("%%d %%d\\n", p != nullptr, given);
""" % (free, padding)
    assert run(tmp_path, body) == [want]
