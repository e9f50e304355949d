"""The host rules that choose a launch form by sizes, compiled from the kernel sources:
the form is the one that measured faster on lattices where the other one had been taken."""
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(__file__), "..", "paper_2504_08157_amd", "csrc")


def _cut(name, start, end):
    src = open(os.path.join(CSRC, name)).read()
    i = src.index(start)
    return src[i:src.index(end, i) + len(end)]


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    d = tmp_path_factory.mktemp("rules")
    text = "\n".join([
        "#include <cstdio>", "#include <cstdlib>", "constexpr int kMaxN = 6, kColElems = 16;",
        _cut("nh_internal.h", "constexpr int kGmresRegM =", ";"), _cut("nh_internal.h", "constexpr int kGmresColM =", ";"),
        _cut("nh_internal.h", "constexpr int kGmresRegSlots =", ";"),
        "struct HeviParams { int nx, ny, nz, N; }; struct GmresArgs { int restart, schur; };",
        _cut("nh_kernels.hip", "#define NH_SPLIT_CASES(X)", "X(6, 4, 1, 2, 2, 3, 1, 1, 1)") + "\n",
        _cut("nh_kernels.hip", "void stage_plan(int N, int nx, int ny, int nelz, int *shape, int *nchunk)\n{", "\n}\n"),
        _cut("nh_colgmres.hip", "bool gmres_lanes_ok(const HeviParams &h, const GmresArgs &g)\n{", "\n}\n"),
        """int main(int argc, char **argv)
{
    int a[8];
    for (int i = 0; i < 6; ++i) a[i] = atoi(argv[i + 2]);
    if (argv[1][0] == 'p') {
        int s, z;
        stage_plan(a[0], a[1] * a[0], a[2] * a[0], a[3], &s, &z);
        printf("%d %d\\n", s, z);
    } else {
        const HeviParams h = {a[1] * a[0], a[2] * a[0], a[3] * a[0] + 1, a[0]};
        printf("%d\\n", (int)gmres_lanes_ok(h, GmresArgs{a[4], a[5]}));
    }
}
"""])
    (d / "rules.cpp").write_text(text)
    exe = str(d / "rules")
    subprocess.run(["g++", "-std=c++17", "-O1", "-o", exe, str(d / "rules.cpp")], check=True)

    def ask(*a):
        return tuple(int(v) for v in subprocess.run([exe] + [str(v) for v in a], check=True, capture_output=True,
                                                    text=True).stdout.split())
    return ask


# order, elements; whole columns of shape 0 against the plan in the comment, us in FP64 / FP32-mixed
@pytest.mark.parametrize("N,nel", [(5, (24, 36, 3)),     # three runs: 25.8, 21.7 against 27.4, 24.1
                                   (3, (118, 34, 7)),    # seven runs: 45.6, 37.9 against 49.3, 44.7
                                   (3, (59, 87, 8)),     # four runs: 51.9, 43.0 against 56.4, 49.8
                                   (2, (154, 79, 2)),    # shape 2, two runs: 10.6, 10.5 against 11.8, 10.9
                                   (4, (128, 128, 20))])
def test_stage_takes_whole_columns(rules, N, nel):
    assert rules("p", N, *nel, 0, 0) == (0, 1)


# the plan taken, its times and those of whole columns of shape 0
@pytest.mark.parametrize("N,nel,plan", [(4, (4, 4, 4), (3, 4)),       # 11 against 27
                                        (4, (40, 40, 16), (0, 2)),    # 58 against 100
                                        (5, (40, 40, 16), (2, 1)),    # 168 against 251
                                        (6, (4, 140, 8), (0, 3))])    # 68 against 77 (79 with eight runs)
def test_stage_splits_where_it_gains(rules, N, nel, plan):
    got = rules("p", N, *nel, 0, 0)
    assert got != (0, 1) and (N == 4 and nel[0] == 4 or got == plan), got


# order, elements, restart, Schur form, elements on lanes; times on lanes and with a column per wave, us
@pytest.mark.parametrize("N,nel,restart,schur,lanes", [
    (6, (26, 26, 3), 10, 0, 0),      # 566 against 383
    (5, (32, 32, 1), 20, 0, 0),      # 549 (390 with the shorter least-squares problem) against 255
    (4, (40, 40, 1), 20, 0, 0),      # 335 (253) against 217
    (4, (2, 2, 4), 10, 0, 0),        # 51 against 43
    (5, (5, 5, 8), 10, 0, 0),
    (4, (40, 40, 12), 10, 0, 1),     # 352 against 720
    (4, (40, 40, 12), 20, 0, 1),     # 847 against 4011
    (5, (30, 30, 16), 10, 1, 1),     # 263 against 882
    (6, (12, 12, 16), 10, 0, 1),     # 517 against 2976
    (4, (40, 40, 17), 10, 0, 0), (4, (40, 40, 12), 21, 0, 0)])
def test_column_solve_form(rules, N, nel, restart, schur, lanes):
    assert rules("c", N, *nel, restart, schur) == (lanes,)
