"""The limits of `csrc/limits.hpp`, compiled by themselves with the host compiler (no GPU)."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2003_10579_amd", "csrc")


def _evaluate(tmp_path, body):
    """Runs `body`, C++ statements that print numbers, against the header."""
    if shutil.which("g++") is None:
        pytest.skip("g++ not available")
    src, exe = tmp_path / "limits.cpp", tmp_path / "limits"
    src.write_text('#include <cstdio>\n#include "limits.hpp"\nusing namespace ssgd;\nint main() {\n' + body + "\nreturn 0;\n}\n")
    subprocess.run(["g++", "-std=c++17", "-Wall", "-Werror", "-I", CSRC, str(src), "-o", str(exe)], check=True)
    out = subprocess.run([str(exe)], check=True, capture_output=True, text=True).stdout
    return [int(v) for v in out.split()]


def test_lanes_that_read_zeros_are_past_every_accepted_matrix(tmp_path):
    """A raw buffer load is out of range from vector offset >= size - scalar offset on.  Sizes on both sides of 2 GiB and of
    the limit; the scalar offset is that of any row, so the first row (offset 0) is the one that asks for most."""
    sizes = [(4096, 64), (700_000, 785), (6_000_000, 100), (536_870_912, 1), (536_870_913, 1), (1_073_741_820, 1), (1_073_741_821, 1),
             (268_435_455, 4), (268_435_456, 4), (2 ** 32 - 1, 3)]
    body = 'printf("%u\\n", kPastMatrix);\n' + "".join(f'printf("%d\\n", (int)one_descriptor_spans({n}ull, {d}ull));\n' for n, d in sizes)
    past, *spans = _evaluate(tmp_path, body)
    assert past % 4 == 0 and past + 16 <= 2 ** 32       # the four words of a load do not wrap
    for (n, d), ok in zip(sizes, spans):
        assert ok == (4 * n * d <= past), (n, d)
        if ok:
            assert past >= 4 * n * d                    # out of range beside row 0, hence beside every row
    assert spans == [1, 1, 1, 1, 1, 1, 0, 1, 0, 0]


def test_schedule_launches_stay_below_the_largest_grid(tmp_path):
    """Work items of one dimension of a launch are counted in 32 bits."""
    per, blocks, block = _evaluate(tmp_path, 'printf("%lld %u %d\\n", (long long)kSyncUpdatesPerLaunch, sync_schedule_blocks(kSyncUpdatesPerLaunch), 64 * kSyncWaves);')
    assert 0 < blocks * block < 2 ** 32 and blocks * block >= 64 * per


def test_clusters_of_four_launches_cannot_keep_each_other_incomplete(tmp_path):
    """Widths up to a whole XCD of 32 CUs: four launches that each hold all but one of the CUs of a cluster leave one free."""
    ok = _evaluate(tmp_path, "".join(f'printf("%d\\n", (int)whole_cus({G}, 256));\n' for G in range(1, 33)))
    assert ok == [1 if G == 1 or 4 * (G - 1) < 32 else 0 for G in range(1, 33)] and ok[:8] == [1] * 8 and not any(ok[8:])


def test_teams_leave_room_for_the_schedule_and_for_other_launches(tmp_path):
    """Every team over a range of shapes and CU counts: a CU per workgroup and one per XCD free; on one XCD four teams that each hold
    all but one of their places leave one; spread over XCDs, where a launch can hold all of its places on one XCD and wait for
    another, four whole launches fit; a member has a tile; alone where there is one tile or no room."""
    cases = [(t, G, C, R, 8 * room, per_cu) for t in (1, 2, 3, 7, 32, 64, 256) for G in (1, 2, 3, 4, 7, 9, 10, 12, 16, 40) for C in (1, 10, 15)
             for R in (1, 2, 7, 8, 9, 40, 300) for room in (10, 31, 32, 33, 38, 40) for per_cu in (1, 2)]
    body = "TeamShape t;\n" + "".join(f't = team_shape({t}, {G}, {C}, {R}, {cus}, {p}); printf("%d %d\\n", t.members, t.spread);\n' for t, G, C, R, cus, p in cases)
    got = _evaluate(tmp_path, body)
    local = wide = 0
    for (t, G, C, R, cus, per_cu), members, spread in zip(cases, got[::2], got[1::2]):
        assert 1 <= members <= max(1, t)
        if members == 1:
            assert not spread
            continue
        room = cus // 8
        places = room * per_cu
        on_xcd = -(-R * members // 8) * G if spread else -(-R // 8) * G * members
        assert on_xcd <= room - 1
        if spread:
            wide += 1
            assert 4 * on_xcd <= places, (t, G, C, R, cus, per_cu)
        else:
            local += 1
            assert 4 * (G * members - 1) < places
    assert local > 100 and wide > 100
    assert got[:2] == [1, 0]
    whole = _evaluate(tmp_path, "".join(f'printf("%d\\n", (int)whole_cus_spread({n}, {8 * room}));\n' for room in (31, 32, 38) for n in range(1, 13)))
    assert whole == [int(4 * n <= room) for room in (31, 32, 38) for n in range(1, 13)]


def test_a_team_goes_on_only_where_its_workgroups_share_the_l2_they_exchange_through(tmp_path):
    """XCDs of the workgroups of made-up placements, [member][slice]: a team that is not spread sits on one XCD as a whole, one that
    is has every cluster on one."""
    cases = [(3, 1, [2, 2, 2]), (3, 1, [2, 2, 5]), (3, 1, [5, 2, 2]), (2, 4, [1] * 8), (2, 4, [1] * 4 + [6] * 4), (2, 4, [1] * 7 + [6]),
             (2, 4, [1, 1, 6, 1] + [1] * 4), (2, 4, [6] + [1] * 7), (1, 3, [0, 0, 0]), (1, 3, [0, 0, 7]), (32, 1, list(range(8)) * 4)]
    body = "".join("{ const int ids[] = {%s}; auto id = [&](int q) { return ids[q]; };\n"
                   'printf("%%d %%d\\n", (int)team_shares_l2(%d, %d, false, id), (int)team_shares_l2(%d, %d, true, id)); }\n'
                   % (", ".join(map(str, ids)), w, G, w, G) for w, G, ids in cases)
    got = _evaluate(tmp_path, body)
    for (w, G, ids), local, spread in zip(cases, got[::2], got[1::2]):
        clusters = [set(ids[G * q:G * q + G]) for q in range(w)]
        assert local == (len(set(ids)) == 1), ids
        assert spread == all(len(c) == 1 for c in clusters), ids


def test_everyone_sees_the_same_end_of_a_team_meeting(tmp_path):
    """All interleavings of workgroups that arrive, look at the count and, after waiting too long, try to close the meeting they saw
    incomplete: nobody goes on as a team while another takes the meeting to be off, a team has everyone, and nobody waits for ever."""
    all_ = 3
    closed = 1 << 31
    words = [n | c for n in range(all_ + 1) for c in (0, closed)]
    table = dict(zip(words, _evaluate(tmp_path, "".join(f'printf("%d\\n", (int)meeting({w}u, {all_}u));\n' for w in words))))
    OPEN, TEAM = 0, 1
    start = (0, (("out", None),) * all_)
    reached, todo, ends = {start}, [start], set()
    while todo:
        word, groups = todo.pop()
        said = {what for state, what in groups if state == "done"}
        assert len(said) <= 1 and (TEAM not in said or all(state != "out" for state, _ in groups)), groups
        if all(state == "done" for state, _ in groups):
            ends |= said
        for i, (state, what) in enumerate(groups):
            nexts = []
            if state == "out":
                nexts.append((word + 1, ("in", None)))
            elif state == "in":
                nexts.append((word, ("in", word) if table[word] == OPEN else ("done", table[word])))
                if what is not None:                                      # the compare-and-swap of the count seen last
                    nexts.append((word | closed if word == what else word, ("in", None)))
            for w, g in nexts:
                new = (w, groups[:i] + (g,) + groups[i + 1:])
                if new not in reached:
                    reached.add(new)
                    todo.append(new)
    assert ends == {1, 2}


def test_launches_of_a_team_are_bounded(tmp_path):
    """At least one update and, from two on, no more tiles of a member than the limit."""
    cases = [(t, w) for t in (1, 2, 3, 9, 64, 1000, 16384, 16385, 65536, 64 * 1024) for w in (2, 3, 8, 32)]
    most, *got = _evaluate(tmp_path, 'printf("%lld\\n", (long long)kTeamTilesPerLaunch);\n' + "".join(f'printf("%lld\\n", (long long)team_updates_per_launch({t}, {w}));\n' for t, w in cases))
    for (t, w), n in zip(cases, got):
        turns = -(-t // w)
        assert n >= 1 and (n == 1 or n * turns <= most) and (n + 1) * turns > most
