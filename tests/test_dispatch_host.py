"""Host side of the launches (CPU only): the library's host code is compiled
without device code, and a small program calls its work-list functions on
hand-made contexts and prints what they decide."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include "qnsch_lib.hip"

// workgroups that each item of a list owns (a workgroup works for the last item
// that starts at or before it) against those it has work for
static void list_case(const char *name, int kind, int precision, int items)
{
    qnsch_ctx x;
    x.g = {};
    x.nlev = 1;
    x.L[0].m1 = x.L[0].pitch = 8;
    x.L[0].m2 = 4;
    x.opt.precision = precision;
    x.lds_max = 163840;
    ItemList W;
    for (int k = 0; k < items; k++) add_item(W, &x, kind, 0);
    for (int k = 0; k < items; k++)
        printf("list %s %d %d %d\n", name, items, W.it.start[k + 1] - W.it.start[k], op_blocks(&x, kind, 0));
    printf("list %s %d %d %d\n", name, items, W.blocks - W.it.start[items - 1], op_blocks(&x, kind, 0));
}

int main()
{
    for (int n : { 1, 2, 3, 12, MAXITEMS }) {
        list_case("bottom", OP_COARSE, QNSCH_FP64, n);
        list_case("mx_bottom", OP_MXCOARSE, QNSCH_MIXED, n);
    }
    return 0;
}
"""


@pytest.fixture(scope="module")
def lines(tmp_path_factory):
    d = tmp_path_factory.mktemp("dispatch")
    src, exe = d / "dispatch.hip", d / "dispatch"
    src.write_text(PROGRAM)
    # host pass only: the kernels' code object is left out, and with it the
    # symbol that the (never used) kernel registration refers to
    subprocess.run(["hipcc", "--offload-host-only", "-O0", "-std=c++17", "-w",
                    "-I", os.path.join(ROOT, "paper_1703_06606_amd", "csrc"), "-I", os.path.join(ROOT, "include"),
                    "-Wl,--unresolved-symbols=ignore-in-object-files", str(src), "-o", str(exe)],
                   check=True, timeout=300)
    out = subprocess.run([str(exe)], check=True, timeout=60, capture_output=True, text=True).stdout
    return [l.split() for l in out.splitlines()]


@pytest.mark.parametrize("kernel", ["bottom", "mx_bottom"])
def test_one_workgroup_per_item_of_the_bottom_levels(lines, kernel):
    """The bottom levels of a cycle are one workgroup's work, in place: an item
    of a list that owned a second workgroup would run its cycle twice, at the
    same time, on the same arrays."""
    rows = [l for l in lines if l[:2] == ["list", kernel]]
    assert len(rows) == sum((1, 2, 3, 12, 64)) + 5
    for r in rows:
        assert int(r[3]) == int(r[4]) == 1, r
