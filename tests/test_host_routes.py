"""Where the dense products of a layer call on a large graph go, on the host: tests/host_routes.cpp writes down what the library launches."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PKG = os.path.join(ROOT, "paper_2212_05009_amd")


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    if not os.path.exists(os.path.join(PKG, "libgcn.so")):
        import __graft_entry__
        __graft_entry__.build()
    out = str(tmp_path_factory.mktemp("host") / "host_routes")
    cmd = [os.environ.get("HIPCC", "/opt/rocm/bin/hipcc"), "-x", "hip", "--offload-host-only", "--offload-arch=gfx950", "-std=c++17", "-O1", "-I", os.path.join(PKG, "csrc"),
           os.path.join(ROOT, "tests", "host_routes.cpp"), "-o", out, "-L", PKG, "-lgcn", "-Wl,-rpath," + PKG, "-rdynamic", "-pthread"]
    res = subprocess.run(cmd, capture_output=True, text=True)
    assert res.returncode == 0, res.stdout + res.stderr
    return out


def dense(program, overlap, call, d_in, d_out, ld, *rows):
    """The launches of dense kernels: (kernel's name, workgroups, stream)."""
    res = subprocess.run([program, str(overlap), call, str(d_in), str(d_out), str(ld), *map(str, rows)], capture_output=True, text=True, timeout=60)
    assert res.returncode == 0, res.stdout + res.stderr
    launches = [line.split() for line in res.stdout.splitlines()]
    return [(k, int(g), s) for k, g, s in launches if "gemm" in k]


CUS = 64        # compute units of a dense product beside a sparse one (GCN_OVERLAP_CUS)


# The forward pass keeps the rounding of the fp32 pipe (hidden values next to zero keep their sign), beside a sparse product, behind one, or alone.
@pytest.mark.parametrize("overlap", [0, 1])
@pytest.mark.parametrize("call,d_in,d_out,ld,rows", [("fwd", 100, 173, 100, []), ("fwd", 201, 256, 201, []), ("fwd", 96, 130, 96, []), ("fwd", 602, 128, 602, []),
                                                     ("fwd", 256, 256, 256, []), ("dense", 602, 128, 602, [232965]), ("dense", 256, 256, 256, [500000]),
                                                     ("dense", 300, 256, 300, [1 << 18]), ("dense", 600, 400, 600, [1 << 18])])
def test_forward_products_are_not_in_three_parts(program, overlap, call, d_in, d_out, ld, rows):
    launches = dense(program, overlap, call, d_in, d_out, ld, *rows)
    assert launches and not any("split" in k for k, _, _ in launches), launches


@pytest.mark.parametrize("d_in,d_out", [(256, 256), (100, 256), (128, 192)])
def test_a_forward_product_that_follows_keeps_to_its_compute_units(program, d_in, d_out):
    launches = dense(program, 1, "fwd", d_in, d_out, d_in)
    assert len(launches) > 1 and all("k_gemm_nn_regw" in k and s == "side" for k, _, s in launches), launches
    assert all(g <= CUS for _, g, _ in launches[:-1]), launches             # (the last has nothing beside it)
    alone = dense(program, 0, "fwd", d_in, d_out, d_in)
    assert {k for k, _, _ in alone} == {k for k, _, _ in launches}, (alone, launches)


# A saved A^ H in rows of odd pitch: the gradient runs behind the sparse product, on the whole chip, in three parts; else beside it on its own units.
@pytest.mark.parametrize("d_in,d_out,ld,apart", [(173, 128, 173, True), (101, 256, 101, True), (128, 101, 129, True), (256, 256, 256, False),
                                                 (100, 256, 100, False), (256, 100, 256, False)])
def test_a_gradient_is_beside_the_sparse_product_only_on_its_own_compute_units(program, d_in, d_out, ld, apart):
    launches = [x for x in dense(program, 1, "bwd", d_in, d_out, ld) if "gemm_tn" in x[0]]
    alone = [x for x in dense(program, 0, "bwd", d_in, d_out, ld) if "gemm_tn" in x[0]]
    assert [k for k, _, _ in launches] == [k for k, _, _ in alone], (launches, alone)
    main = [x for x in launches if "reduce" not in x[0] and "finish" not in x[0] and "sum" not in x[0]]
    assert len(main) == 1, launches
    assert ("k_gemm_tn_split" in main[0][0]) == apart, launches
    assert main[0][2] == ("main" if apart else "side"), launches
    assert apart or main[0][1] <= CUS, launches


# Sizes from which the three-part kernels were measured to gain: on both sides of the lines, and where they never do.
@pytest.mark.parametrize("terms,columns,rows,split,masked", [
    (256, 256, 1 << 16, True, True), (256, 256, (1 << 16) - 1, False, False), (128, 192, 1 << 16, True, True), (100, 256, 500000, False, False),
    (101, 256, 500000, False, False), (61, 256, 1 << 16, True, False), (61, 256, (1 << 16) - 1, False, False), (47, 256, 500000, False, False),
    (128, 128, 500000, False, False), (300, 41, 1 << 16, True, True), (300, 41, 1 << 15, False, False), (300, 64, 20000, True, True), (368, 173, 8193, True, True),
    (368, 173, 8191, False, False), (300, 256, 1 << 15, True, True), (300, 256, (1 << 15) - 1, False, False), (600, 400, 1 << 14, True, True),
    (600, 400, 9000, False, False), (237, 100, 65, True, True), (237, 100, 64, False, False), (300, 64, 8191, False, False), (300, 64, 8192, True, True),
    (237, 64, 65, True, True), (602, 100, 1, True, True)])
def test_sizes_of_products_in_three_parts(program, terms, columns, rows, split, masked):
    for call, want in (("down", split), ("masked", masked if columns > terms else split)):       # (else the sparse product is last, and takes the mask)
        launches = [k for k, _, _ in dense(program, 1, call, columns, terms, columns, rows) if "gemm_nn" in k]
        assert len(launches) == 1 and ("k_gemm_nn_split" in launches[0]) == want, (call, launches)


@pytest.mark.parametrize("d_in,d_out,rows,split", [(256, 256, 2048, True), (256, 256, 2047, False), (80, 200, 2048, True), (72, 72, 20000, False), (72, 72, 1 << 17, True),
                                                   (128, 128, 1 << 16, False), (128, 128, 100000, True), (384, 128, 1 << 14, False), (384, 128, 1 << 15, True),
                                                   (128, 66, 2048, True), (65, 65, 1 << 16, False), (65, 65, 1 << 17, True), (173, 128, 1 << 15, False),
                                                   (602, 128, 8192, False), (602, 128, 20000, True), (128, 64, 500000, False)])
def test_sizes_of_gradients_in_three_parts(program, d_in, d_out, rows, split):
    launches = [k for k, _, _ in dense(program, 1, "grad", d_in, d_out, d_in, rows) if "gemm_tn" in k]
    assert any("k_gemm_tn_split" in k for k in launches) == split, launches
