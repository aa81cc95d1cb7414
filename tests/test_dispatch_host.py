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

// the smoothing launches, transfers and buffers of a cycle
static void cycle_case(int m1, int m2, int bcx, int bcy, int nu1, int nu2, int precision)
{
    qnsch_ctx x;
    x.g = {};
    x.g.bc_x = bcx;
    x.g.bc_y = bcy;
    qnsch_default_opts(&x.opt);
    x.opt.nu1 = nu1;
    x.opt.nu2 = nu2;
    x.opt.precision = precision;
    x.lds_max = 163840;
    x.ncu = 256;
    for (; x.nlev < 3; x.nlev++) {
        DLev &D = x.L[x.nlev];
        D.m1 = D.pitch = m1 >> x.nlev;
        D.m2 = m2 >> x.nlev;
    }
    std::vector<Op> prog;
    cycle_program(&x, prog);
    printf("cycle %d %d %d %d %d %d", m1, m2, bcx, bcy, nu1, nu2);
    for (const Op &o : prog) {
        const char *k = "other";
        if (o.kind == OP_HS || o.kind == OP_MXHS) k = "half";
        if (o.kind == OP_FUSED || o.kind == OP_MXFUSED) k = o.colour & FUSED_TWO ? "two" : "one";
        if (o.kind == OP_RESTRICT || o.kind == OP_MXRESTRICT) k = "restrict";
        if (o.kind == OP_PROLONG || o.kind == OP_MXPROLONG) k = "prolong";
        if (o.kind == OP_COARSE || o.kind == OP_MXCOARSE) k = "bottom";
        printf(" %s:%d:%d", k, o.level, k[0] == 't' || k[0] == 'o' ? o.colour & 3 : o.colour);
    }
    printf("\n");
}

int main()
{
    for (int precision : { QNSCH_FP64, QNSCH_MIXED })
        for (int nu1 = 0; nu1 <= 6; nu1++)
            for (int nu2 = 0; nu2 <= 6; nu2++) {
                cycle_case(16, 16, 1, 1, nu1, nu2, precision);
                cycle_case(16, 64, 1, 0, nu1, nu2, precision);
                cycle_case(64, 16, 0, 1, nu1, nu2, precision);
                cycle_case(16, 16, 0, 0, nu1, nu2, precision);
                cycle_case(20, 24, 1, 1, nu1, nu2, precision);
                cycle_case(12, 40, 1, 0, nu1, nu2, precision);
                cycle_case(160, 128, 1, 1, nu1, nu2, precision);
            }
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


def test_smoothing_launches_of_a_cycle(lines):
    """Every level's nu1 and nu2 sweeps are launched, each launch reads the set of
    cell unknowns that the one before it left, the cycle ends in the first set,
    and a fused launch is used only where the periodic axes are as long as its
    widened tile asks for: 19 cells with one sweep, 15 with two."""
    rows = [l for l in lines if l[0] == "cycle"]
    assert len(rows) == 2 * 49 * 7
    twos = 0
    for r in rows:
        m1, m2, bcx, bcy, nu1, nu2 = (int(v) for v in r[1:7])
        ops = [(k, int(l), int(c)) for k, l, c in (o.split(":") for o in r[7:])]
        bottom = next(l for k, l, c in ops if k == "bottom")
        cells, face, sweeps, phase = {}, {}, {}, 0
        for k, l, c in ops:
            dims = [m >> l for m, per in ((m1, bcx), (m2, bcy)) if per]
            cur = cells.get(l, 0)
            if k in ("one", "two"):
                assert min(dims, default=99) >= (19 if k == "one" else 15), (r[1:7], k, l)
                assert c & 1 == cur and (c < 2 or phase == 1), (r[1:7], k, l)
                cells[l] = cur ^ 1
                face[l] = face.get(l, 0) ^ 1
                sweeps[l, phase] = sweeps.get((l, phase), 0) + (1 if k == "one" else 2)
                twos += k == "two"
            elif k == "half":
                assert cur == 0, (r[1:7], k, l)
                face[l] = face.get(l, 0) ^ 1
                sweeps[l, phase] = sweeps.get((l, phase), 0) + 0.5
            elif k == "restrict":
                assert c == cur, (r[1:7], k, l)
            elif k == "prolong":
                assert cur == 0, (r[1:7], k, l)
            elif k == "bottom":
                phase = 1
        assert not any(cells.values()) and not any(face.values()), r[1:7]
        for l in range(bottom):
            assert sweeps.get((l, 0), 0) == nu1 and sweeps.get((l, 1), 0) == nu2, (r[1:7], l)
            corrected = [k for k, lev, c in ops if lev == l and (k == "prolong" or (k in ("one", "two") and c & 2))]
            assert len(corrected) == 1, (r[1:7], l)
    assert twos > 0
