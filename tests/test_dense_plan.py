"""How a dense pass is cut into workgroups (no GPU needed): `dense_stream_plan`, asked by a small host program.

Whatever the sizes: the launches cover every member once and every row, a group's members share one block of the random
stream, the kernel for the group's size exists, and the reproducible mode gets the one layout that it can order.  And the
sizes that the GPU test of single products runs at reach every kernel that a plan can name."""
import itertools
import os
import subprocess

import pytest

SOURCE = r"""
#include "kernels.h"
#include <cstdio>
using namespace nnr;
int main() {
  long n;
  int m, k, q, perturb, ordered;
  while (scanf("%ld %d %d %d %d %d", &n, &m, &k, &q, &perturb, &ordered) == 6) {
    Dims d{};
    d.n = n; d.n_pad = (n + 255) / 256 * 256; d.m = m; d.k = k; d.kp = (k + 15) / 16 * 16; d.q = q;
    const DensePlan p = dense_stream_plan(d, perturb != 0, ordered != 0);
    printf("%d %d", p.full_members, p.tail_members);
    for (const StreamPart& s : p.part) printf(" %d %d %d %ld", s.waves, s.members, s.groups, (long)s.chunks);
    printf("\n");
  }
}
"""


@pytest.fixture(scope="module")
def plans(tmp_path_factory):
    from paper_2202_09512_amd import build
    objs = [os.path.join(build.HERE, "_build", f) for f in ("kernels_dense.o", "kernels_small.o")]
    if not all(os.path.exists(o) for o in objs):
        build.build(verbose=False)
    folder = tmp_path_factory.mktemp("dense_plan")
    src, exe = folder / "plan.cpp", folder / "plan"
    src.write_text(SOURCE)
    subprocess.run(["/opt/rocm/bin/hipcc", "-std=c++17", "-O1", "-x", "c++", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-I",
                    os.path.join(build.HERE, "csrc"), str(src), "-x", "none", *objs, "-o", str(exe)], check=True)

    def ask(sizes):
        text = "".join("%d %d %d %d %d %d\n" % tuple(s) for s in sizes)
        out = subprocess.run([str(exe)], input=text, check=True, capture_output=True, text=True, timeout=120).stdout
        rows = [[int(v) for v in line.split()] for line in out.splitlines()]
        assert len(rows) == len(sizes)
        # (full members, tail members, [(waves, members, groups, chunks) of the two launches])
        return [(r[0], r[1], [tuple(r[2:6]), tuple(r[6:10])]) for r in rows]
    return ask


def test_plans_cover_members_and_rows(plans):
    sizes = list(itertools.product(
        (1, 2, 15, 16, 17, 63, 64, 65, 127, 128, 129, 300, 1000, 2049, 7001, 16384, 40000), (1, 3, 40), (1, 16, 17, 32, 33, 48, 64),
        (1, 2, 3, 4, 5, 7, 8, 9, 15, 16, 20, 63, 64), (0, 1), (0, 1)))
    for (n, m, k, q, perturb, ordered), (full, tail, parts) in zip(sizes, plans(sizes)):
        nt, where = (k + 15) // 16, (n, m, k, q, perturb, ordered)
        assert full + tail == q, where
        for first, count, (waves, members, groups, chunks) in ((0, full, parts[0]), (full, tail, parts[1])):
            assert (groups > 0) == (count > 0), where
            if not groups:
                continue
            # members [first + g * members, ...): all covered, by groups that lie inside one block of eight draws; the slots
            # past the ensemble's end are at most the seven that the operand array has to spare
            assert members in (1, 2, 4, 8) and members * nt <= 8 and first % members == 0, where
            assert count <= members * groups < count + members, where
            assert waves == 8 or (waves == 4 and not ordered and members * nt <= max(2, nt)), where
            rows = -(-n // chunks)
            rows = -(-rows // (16 * waves)) * 16 * waves          # rows of a chunk, as the launch rounds them
            assert chunks >= 1 and -(-n // rows) == chunks, where
            assert not ordered or chunks == 1, where
            assert -(-n // (16 * waves)) * m * groups * chunks <= 0x7FFFFFFF, where


def test_sizes_of_the_single_product_test_reach_every_kernel(plans):
    from tests.test_gpu_dense_terms import FORMS
    for perturb in (0, 1):
        reached, tails = set(), set()
        for (n, k, q), (full, tail, parts) in zip(FORMS, plans([(n, 1, k, q, perturb, 0) for n, k, q in FORMS])):
            nt = (k + 15) // 16
            for waves, members, groups, _ in parts:
                if groups:
                    reached.add((nt, waves, members))
            if full and tail:
                tails.add((nt, parts[1][1]))
        every = {(nt, 8, g) for nt in (1, 2, 3, 4) for g in (1, 2, 4, 8) if g * nt <= 8}
        every |= {(nt, 4, g) for nt in (1, 2, 3, 4) for g in (1, 2) if g * nt <= max(2, nt)}
        assert reached == every, (perturb, every - reached, reached - every)
        assert tails == {(1, 1), (1, 2), (1, 4), (2, 1), (2, 2), (3, 1), (4, 1)} or not perturb, tails
