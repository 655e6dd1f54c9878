"""The profile summarizer of bench.py on launches whose lanes do not name their
workload (no GPU): steps in strips, steps that several blocks share and steps on
flat row groups are listed under the workload of the launch before them."""
import bench

NS = "lbm::(anonymous namespace)::"


def _launch(n, kernel, model, prec, grid, *flags):
    args = [f"lbm::{model}", f"{NS}{prec}"] + [("true" if f else "false") for f in flags]
    return {"Dispatch_Id": str(n), "Grid": grid,
            "Kernel_Name": f"void {NS}{kernel}<{', '.join(args)}>({NS}{prec}::S const*)"}


def test_launches_without_a_workload_of_their_own_take_the_one_before():
    cells3, cells2 = 11 * 11 * 800, 11 * 800
    rows = [_launch(1, "k_init", "D3Q95", "F32ST", -(-cells3 // 256) * 256),
            _launch(2, "k_step", "D3Q95", "F32ST", 1600 * 64, 1, 0, 0, 1, 1),      # flat groups
            _launch(3, "k_step_split", "D3Q95", "F32ST", 4 * cells3, 0),
            _launch(4, "k_init", "D2Q33", "F64T", -(-cells2 // 256) * 256),
            _launch(5, "k_steps_strip", "D2Q33", "F64T", 200 * 320, 1)]
    got = [(inst, label, cells, alg) for _, inst, label, cells, alg in
           bench._walk_dispatches(rows, lambda r: r["Grid"])]
    assert got[1] == ("k_step<D3Q95,F32S,0,1,1>", "11x11x800", cells3, 760 * cells3)
    assert got[2] == ("k_step_split<D3Q95,F32S,0>", "11x11x800", cells3, 760 * cells3)
    assert got[4] == ("k_steps_strip<D2Q33,F64,1>", "11x800", cells2, 528 * cells2)
