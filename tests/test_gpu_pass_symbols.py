"""Which kernel function runs each pass (pf_pass_symbol), for every length with a
compile-time mixed-radix plan in each role, both precisions and (Z) both layouts:
the mixed-radix kernels, but for the power-of-two X lengths 512 and 1024, C2C 512 and
1024, and FP64 C2C 256 beside a power-of-two X pass; the runtime-radix kernels for
343, 686, lengths below 16 and the Chebyshev and empty third transforms.
"""
import pytest

import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
import paper_1905_02803_amd as pf  # noqa: E402

F, B = pf.PF_DIR_FORWARD, pf.PF_DIR_BACKWARD


def symbols(plan):
    return {plan.pass_name(d, i): plan.pass_symbol(d, i) for d in (F, B) for i in range(plan.num_passes(d))}


@pytest.mark.parametrize("f64", [False, True], ids=["f32", "f64"])
def test_every_length_in_every_role(f64):
    d = "d" if f64 else ""
    for n in synth.smooth7(16, 1024):
        x, c = ("k_mr_x", "k_mr_x"), "k_mr_c2c"
        if n in (512, 1024):
            x, c = ("k_r2c_p2" + d, "k_c2r_p2" + d), "k_c2c_p2" + d
        elif n in (343, 686):
            x, c = ("k_r2c_x", "k_c2r_x"), "k_c2c_tile"
        print(f"case pass symbols {n} f64={f64}", flush=True)
        for (nx, ny, nz), stride1 in (((n, 6, 4), 1), ((8, n, 4), 1), ((8, 4, n), 1), ((8, 4, n), 0)):
            lay = pf.Layout(precision=pf.PF_F64 if f64 else pf.PF_F32, stride1=stride1)
            with pf.Plan(nx, ny, nz, lay) as plan:
                s = symbols(plan)
            rest = {"x": ("k_r2c_x", "k_c2r_x"), "c": "k_c2c_tile"}
            assert (s["fwd_x_r2c"], s["bwd_x_c2r"]) == (x if nx == n else rest["x"]), (nx, ny, nz)
            assert {s["fwd_y_c2c"], s["bwd_y_c2c"]} == {c if ny == n else rest["c"]}, (nx, ny, nz)
            assert {s["fwd_z_c2c"], s["bwd_z_c2c"]} == {c if nz == n else rest["c"]}, (nx, ny, nz)


def test_exceptions():
    with pf.Plan(512, 256, 16, pf.Layout(precision=pf.PF_F64)) as plan:
        assert symbols(plan)["fwd_y_c2c"] == "k_c2c_p2d"
    for third in (pf.PF_THIRD_CHEB, pf.PF_THIRD_EMPTY):
        with pf.Plan(60, 60, 61, pf.Layout(third=third)) as plan:
            s = symbols(plan)
        assert s["fwd_z_c2c"] == "k_c2c_tile" and s["fwd_y_c2c"] == "k_mr_c2c"
    with pf.Plan(60, 60, 60, pf.Layout(m1=2, m2=2)) as plan:
        s = symbols(plan)
        assert s["fwd_pack_x_pencils"] == "k_remap" and s["fwd_x_r2c"] == "k_mr_x"
        assert plan.pass_symbol(F, 99) == ""
