"""The peel's edge classes: edges of at most 64 triangles are taken side by side, of at most 4,096 by a
wave, longer ones by a workgroup.  Levels, ranks and sizes at these lines, and with several long edges
a workgroup in one round, against the oracle."""
import pytest

from test_gpu_peel import book, check, ebb  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("pages", [63, 64, 65, 4095, 4096, 4097])
def test_edges_at_the_lines(ebb, pages):  # noqa: F811
    check(ebb, book(pages), f"book{pages}", pages)
    check(ebb, book(pages, 3), f"3 books of {pages}", 3 * pages)


def test_several_long_edges_a_workgroup(ebb):  # noqa: F811
    # 1.0 M edges on 64 workgroups; the 124 spines leave together in the second round
    check(ebb, book(4097, 124), "124 books", 4097 * 124)
