"""Dense launches whose XCDs take KV groups of their own (csrc/rr_attn_rows.hpp), on the host: every row is taken once, no XCD takes groups
of another, and none has more work than its share but for what the last rows leave.  A row's work is its number of key blocks."""
import os
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2602_05853_amd", "csrc")

PROGRAM = r'''
#include <cstdio>
#include <cstdlib>
#include "rr_attn_rows.hpp"
int main(int argc, char** argv) {
    for (int a = 1; a + 3 < argc; a += 4) {
        const int NG = atoi(argv[a]), G = atoi(argv[a + 1]), Nb = atoi(argv[a + 2]), packed = atoi(argv[a + 3]);
        const int k = NG < 8 ? 8 / NG : 1;
        const int grid = NG < 8 ? 8 * G * ((Nb + k - 1) / k) : NG * G * Nb;
        for (int bid = 0; bid < grid; ++bid) {
            const rr::RowPlace p = NG < 8 ? rr::row_of_shared_group(bid, NG, G, Nb, packed != 0) : packed ? rr::row_of_groups_by_rank(bid, NG, G) : rr::row_of_whole_groups(bid, G, Nb);
            printf("%d %d %d\n", p.grp, p.hl, p.mr);
        }
        printf("end\n");
    }
}
'''

SHAPES = [(NG, G, Nb, packed) for NG in (1, 2, 4, 8, 16) for G in (1, 4, 7, 8, 32) for Nb in (1, 7, 8, 16, 17, 24, 32, 64) for packed in (0, 1)]
PROMPTS = [(NG, G, n0, n1) for NG in (1, 2, 4) for G in (1, 7, 32) for n0, n1 in ((100, 100), (37, 101), (96, 80), (65, 28), (12, 56))]


RULE = r'''
#include <cstdio>
#include <cstdlib>
#include "rr_attn_rows.hpp"
int main(int argc, char** argv) {
    int v[5];
    for (int i = 0; i < 5 && i + 1 < argc; ++i) v[i] = atoi(argv[i + 1]);
    printf("%d\n", (int)rr::dense_order(v[0], v[1], 128, v[2], v[3] != 0, v[4]));
}
'''


GROUPS = r'''
#include <cstdio>
#include <cstdlib>
#include "rr_attn_rows.hpp"
int main(int argc, char** argv) {
    int v[5];
    for (int i = 0; i < 5 && i + 1 < argc; ++i) v[i] = atoi(argv[i + 1]);
    printf("%d %d\n", rr::rows_by_group(v[0], v[1], v[2], v[3], v[4], 128), rr::front_rows_of_groups(v[2], v[0] / v[2] / (v[4] / 128), v[4] / 128));
}
'''


DECODE = r'''
#include <cstdio>
#include "rr_attn_rows.hpp"
int main() {
    for (int R = 1; R <= 32; ++R)
        for (int parts = 1; parts <= 600; ++parts)
            for (int len = 2; len <= 20; ++len) {
                const rr::DecodeForm f = rr::decode_form(R, parts, len);
                printf("%d %d %d %d %d\n", R, parts, len, f.eight, f.halves);
            }
}
'''


def _compile(d, name, text):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("no C++ compiler")
    (d / f"{name}.cpp").write_text(text)
    subprocess.run([gxx, "-std=c++17", "-Wall", "-Werror", "-I", CSRC, str(d / f"{name}.cpp"), "-o", str(d / name)], check=True)
    return str(d / name)


# KV groups, keys, queries in whole blocks, packed, rows -> sets over all XCDs (0), groups of their own one after the other (1), rank by rank
# (2).  Whole prompts of any length; chunks while the keys and values of the groups in flight are 256 MB at most; numbers of groups
# that do not divide into the XCDs, or the XCDs into them, never.
@pytest.mark.parametrize("NG,L,Lq,packed,rows,order",
                         [(8, 131072, 131072, 0, 32768, 1), (1, 512, 512, 0, 128, 1), (3, 4096, 4096, 0, 1024, 0), (12, 4096, 4096, 0, 1536, 0),
                          (8, 65536, 4096, 0, 1024, 1), (8, 65664, 4096, 0, 1024, 0), (8, 131072, 2048, 0, 512, 0), (16, 65536, 2048, 0, 1024, 1),
                          (16, 80000, 2048, 0, 1024, 0), (4, 131072, 8192, 0, 1792, 1), (4, 131200, 8192, 0, 1792, 0), (1, 600064, 1024, 0, 256, 0),
                          # several groups to an XCD: the last one's heavy rows must not start late
                          (16, 98304, 98304, 0, 24576, 1), (32, 3200, 3200, 0, 800, 2), (32, 1536, 1536, 0, 384, 2), (24, 4224, 4224, 0, 792, 2),
                          (128, 512, 512, 0, 2048, 2), (32, 24064, 24064, 0, 6016, 1), (40, 2560, 2560, 0, 800, 2),
                          # rows of a deep chunk weigh nearly the same
                          (32, 20096, 2176, 0, 544, 1), (64, 3072, 1664, 0, 832, 2), (96, 4096, 384, 0, 288, 2), (64, 12032, 640, 0, 2560, 1),
                          (32, 5120, 5120, 1, 1280, 2), (32, 40960, 40960, 1, 10240, 2), (8, 40960, 40960, 1, 10240, 1)])
def test_order_of_dense_calls(tmp_path, NG, L, Lq, packed, rows, order):
    exe = _compile(tmp_path, "rule", RULE)
    out = subprocess.run([exe, *map(str, (NG, L, Lq, packed, rows))], check=True, capture_output=True, text=True).stdout
    assert int(out) == order


@pytest.fixture(scope="module")
def rows(tmp_path_factory):
    exe = _compile(tmp_path_factory.mktemp("rows"), "rows", PROGRAM)
    wanted = SHAPES + [(NG, G, n0 + n1, 1) for NG, G, n0, n1 in PROMPTS]
    out = subprocess.run([exe] + [str(v) for s in wanted for v in s], check=True, capture_output=True, text=True).stdout
    return {s: [tuple(map(int, line.split())) for line in part.strip().split("\n")]
            for s, part in zip(wanted, out.split("end\n"))}


@pytest.mark.parametrize("NG,G,Nb,packed", SHAPES)
def test_rows_are_taken_once_and_shared_evenly(rows, NG, G, Nb, packed):
    work, seen, groups = [0] * 8, set(), [set() for _ in range(8)]
    for bid, (grp, hl, mr) in enumerate(rows[NG, G, Nb, packed]):
        if mr >= Nb:                                   # the last query blocks of a number that the XCDs do not divide
            continue
        assert 0 <= grp < NG and 0 <= hl < G and mr >= 0
        assert (grp, hl, mr) not in seen
        seen.add((grp, hl, mr))
        work[bid & 7] += Nb - mr
        groups[bid & 7].add(grp)
    assert len(seen) == NG * G * Nb
    for x in range(8):
        assert groups[x] <= {x % NG} if NG < 8 else groups[x] == set(range(x, NG, 8))
    if NG >= 8:
        assert max(work) == min(work)
        return
    # k = 8 / NG XCDs share a group.  A turn is k query blocks of a head that lie side by side, one for each of them.  Two levels of turns
    # taken forth and back leave no difference; a last odd one leaves k - 1 blocks a head at most, one that k does not fill its heaviest
    # row's.  Below two whole levels the place moves on by one from turn to turn: k turns leave none, j < k of them j (k - j) blocks.
    k = 8 // NG
    if Nb < 2 * k:
        bound = sum((n % k) * (k - n % k) for n in (G * (Nb // k), G if Nb % k else 0))
    else:
        bound = G * (k - 1) * (Nb // k % 2) + G * (Nb % k)
    assert max(work) - min(work) <= bound, work


@pytest.mark.parametrize("NG,G,n0,n1", PROMPTS)
def test_two_packed_prompts_are_shared_evenly(rows, NG, G, n0, n1):
    """The weight of a row jumps where a prompt starts: no XCD has the heavy side of that level for more than half of the heads of
    a group beyond another."""
    Nb, k = n0 + n1, 8 // NG
    work = [0] * 8
    for bid, (grp, hl, mr) in enumerate(rows[NG, G, Nb, 1]):
        if mr < Nb:
            m = Nb - 1 - mr
            work[bid & 7] += m + 1 - (n0 if m >= n0 else 0)
    # half of the heads times the jump, and up to k blocks a head in the level that is its partner, in an odd one and in one that k
    # does not fill
    assert max(work) - min(work) <= -(-G // 2) * n0 + 3 * k * G, work


def test_two_workgroups_to_a_part_run_at_once(tmp_path):
    """A second workgroup to a part may not make a second round of the launch: with it there are no more workgroups than compute units (256;
    one of eight waves fills a unit), and parts that fit them one by one still run on eight waves."""
    out = subprocess.run([_compile(tmp_path, "decode", DECODE)], check=True, capture_output=True, text=True).stdout
    taken = 0
    for R, parts, length, eight, halves in (map(int, line.split()) for line in out.strip().split("\n")):
        assert not halves or (R > 16 and 2 * parts <= 256), (R, parts, length)
        assert halves or R <= 16 or 2 * parts > 256, (R, parts, length)
        assert eight == (parts < 256 and length >= 8), (R, parts, length)
        taken += halves
    assert taken


# rows, workgroups at once, KV groups, groups to a set in the other order, keys -> by group; heads of one block each
@pytest.mark.parametrize("rows,resident,NG,interleave,L,own", [(4096, 512, 8, 4, 16384, 1), (4095, 512, 8, 4, 16384, 0), (2048, 512, 16, 8, 8192, 1),
                                                               (2047, 512, 16, 8, 8192, 0), (4096, 512, 32, 8, 8192, 1), (8192, 512, 64, 8, 8192, 1), (16384, 512, 256, 8, 8192, 1), (2048, 256, 2, 2, 33024, 1),
                                                               # queues of one group and of two, of two and of three
                                                               (2268, 512, 9, 3, 8064, 0), (2844, 512, 9, 3, 10112, 0), (4500, 512, 9, 3, 16000, 1),
                                                               (2200, 512, 10, 5, 7040, 0), (2268, 512, 18, 6, 8064, 0), (2304, 512, 18, 9, 4096, 0),
                                                               (2200, 512, 20, 5, 7040, 0), (2244, 512, 11, 1, 13056, 1), (2156, 512, 22, 2, 12544, 1),
                                                               (2125, 512, 17, 1, 16000, 1), (8192, 512, 8, 1, 65536, 0), (8192, 512, 8, 1, 65408, 1)])
def test_rows_that_are_drawn_by_kv_group(tmp_path, rows, resident, NG, interleave, L, own):
    exe = _compile(tmp_path, "groups", GROUPS)
    out = subprocess.run([exe, *map(str, (rows, resident, NG, interleave, L))], check=True, capture_output=True, text=True).stdout.split()
    assert int(out[0]) == own
    # rank by rank throughout where the queues have different numbers of groups: the last of the groups would start late
    G, Nb = rows // NG // (L // 128), L // 128
    # queues of as many groups: sixteen rows a head in all, of each group the same number
    each = 16 // max(NG // 8, 2) or 1
    assert int(out[1]) == (G * Nb if NG > 8 and NG % 8 else (each * G if Nb > each else 0))
