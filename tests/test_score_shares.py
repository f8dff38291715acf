"""How the score sweeps share out the middle tokens (host arithmetic): rounds of workgroups, and the workspace that covers them."""
import os
import subprocess

import pytest

import paper_2502_14477_amd as esa

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LENGTHS = sorted({1, 2, 63, 64, 65, 4661, 5400, 6500, 9300, 10894, 10900, 14500, 16384, 16385, 18500, 18849, 20000, 33000, 60000, 65536, 65537, 130560,
                  130561, 131072, 131073, 140000, 160000, 163841, 190000, 196608, 250000, 262144, 400000, 1000003} | {97 * i for i in range(1, 400)})
BATCHES = [1, 2, 3, 4, 5, 6, 7, 8, 9, 16, 24, 255, 256, 257, 300]
PROGRAM = r"""
#include <cstdio>
#include "score_shares.h"
int main() {
  long long n; int eps, batch;
  while (scanf("%lld %d %d", &n, &eps, &batch) == 3)
    printf("%lld %lld %lld %lld %d\n", (long long)esa::share_tiles(n, eps, batch), (long long)esa::share_count(n, eps, batch),
           (long long)esa::share_rounds(n, eps, batch), (long long)esa::most_shares(n, eps, batch), (int)esa::sweep_pools(n, eps, batch, 16));
}
"""


@pytest.fixture(scope="module")
def shares(tmp_path_factory):
    """{(n, eps, batch): (tiles, shares of a row, rounds, bound of all shares, pooled by the sweep)}"""
    path = tmp_path_factory.mktemp("shares")
    (path / "main.cpp").write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-I", os.path.join(ROOT, "paper_2502_14477_amd", "csrc"), str(path / "main.cpp"), "-o", str(path / "main")], check=True)
    asked = [(n, eps, batch) for n in LENGTHS for eps in (0, 1, 16) for batch in BATCHES]
    out = subprocess.run([str(path / "main")], input="".join("%d %d %d\n" % a for a in asked), capture_output=True, text=True, check=True).stdout
    return dict(zip(asked, (tuple(map(int, line.split())) for line in out.splitlines())))


def test_shares_cover_every_row_in_the_fewest_rounds(shares):
    for (n, eps, batch), (tiles, count, rounds, _, _) in shares.items():
        row = lambda t: -(-n // (32 * t - 2 * eps))
        assert tiles % 2 == 0 and 2 <= tiles <= 16 and count == row(tiles)
        assert rounds == -(-batch * row(16) // 256)                              # what the longest shares need
        assert batch * count <= 256 * rounds                                     # and no workgroup more
        assert tiles == 2 or batch * row(tiles - 2) > 256 * rounds               # in shares no longer than that takes


def test_pooling_in_the_sweep_takes_no_round_more(shares):
    for (n, eps, batch), s in shares.items():
        assert s[4] == (s[2] == shares[n, 0, batch][2])
    assert not shares[131072, 1, 1][4] and shares[130560, 1, 1][4]


def test_bound_of_the_shares_covers_shorter_rows_and_fewer_of_them(shares):
    for eps in (0, 1, 16):
        for i, batch in enumerate(BATCHES):
            most = [shares[n, eps, batch][3] for n in LENGTHS]
            assert most == sorted(most)
            for n in LENGTHS:
                assert shares[n, eps, batch][3] >= batch * shares[n, eps, batch][1]
                assert shares[n, eps, batch][3] >= batch * shares[n, 0, batch][1]          # where a kernel of its own pools
                assert i == 0 or shares[n, eps, batch][3] >= shares[n, eps, BATCHES[i - 1]][3]


def test_row_of_a_share():
    """The quotient as the sweeps find it: exact for shares up to 2^31 - 1, of rows of any length."""
    for n in [1, 2, 3, 5, 7, 255, 256, 257, 1023, 1024, 65537, 10 ** 6, 2 ** 30, 2 ** 31 - 1] + list(range(1, 300, 11)):
        inverse = 0xFFFFFFFF // n                                                 # inverse_of
        top = 2 ** 31 - 1
        for s in sorted({x for q in (0, 1, 2, 1000, 65534, top // n - 1, top // n) for x in (q * n - 1, q * n, q * n + 1, q * n + n - 1, top) if 0 <= x <= top}):
            b = s * inverse >> 32
            assert b + (s - b * n >= n) == s // n, (s, n)


def test_score_workspace_for_the_longest_context_covers_shorter_ones():
    # 512 and 77 queries; rows beyond the size at which S is stored
    for l_c in (512, 77):
        for eps in (0, 1, 16, 40):
            for batch in (1, 3, 7):
                sizes = [esa.lib.esa_score_workspace_bytes(l_c, n, eps, batch) for n in LENGTHS if l_c * n * 4 > 16 << 20]
                assert sizes == sorted(sizes)


@pytest.mark.parametrize("eps", [0, 1, 16, 40])
def test_score_workspace_for_a_chunk_covers_what_follows_it(eps):
    """Shorter chunks, and one token, for any row."""
    for n in LENGTHS:
        for batch in (1, 3, 16):
            for size in (lambda l_c: esa.lib.esa_score_workspace_bytes(l_c, n, eps, batch),
                         lambda l_c: esa.lib.esa_score_select_gather_workspace_bytes(l_c, n, eps, 2048, batch)):
                swept = [l_c for l_c in (17, 20, 32, 77, 300, 512, 513, 1024) if l_c * n * batch * 4 > 16 << 20]
                sizes = [size(l_c) for l_c in swept]
                assert sizes == sorted(sizes)
                assert all(s >= size(1) for s in sizes), (n, batch)
    assert esa.lib.esa_score_workspace_bytes(512, 20000, eps, 1) >= esa.lib.esa_score_workspace_bytes(8, 20000, eps, 1)      # whose scores are stored
