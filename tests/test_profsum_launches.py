"""Names, workgroups and bytes of the launches that sum an FP64 solve's norm, as
they stand in the kernel traces of whole solves (profiles/k_solves_fused_legs_pairs.md),
and the listing of the sweeps by colour under their own name."""

import json
import sqlite3

import pytest

from paper_1406_5369_amd import profsum


def info(form, sweeps, by, waves=8, prefetch=1):
    return dict(form=form, sweeps=sweeps, by=by, zchunk=64, prefetch=prefetch, waves=waves, blocks=1)


def test_leg():
    name, _, needed = profsum.norm_launch(info("leg", 2, 32), 2, 129)
    assert name == "mg::k_down2d<double, 0, 4, 2>"
    # u, f and the iterate on 127^2 inner nodes, the right-hand side on 63^2 coarse ones
    assert needed == 8 * (3 * 127**2 + 63**2)
    assert profsum.norm_launch(info("leg", 1, 64), 2, 4097)[0] == "mg::k_down2d<double, 0, 4, 4>"
    name, _, needed = profsum.norm_launch(info("leg", 2, 32), 2, 129, var=True)
    assert name == "mg::k_down2d<double, 1, 4, 2>" and needed == 8 * (4 * 127**2 + 63**2)


def test_pair_and_sweep():
    name, note, needed = profsum.norm_launch(info("pair", 2, 32), 3, 257)
    assert name == "mg::k_smooth3d_x2<double, 0, 2, 8, 4>" and needed == 24 * 255**3 and "two" in note
    name, _, needed = profsum.norm_launch(info("sweep", 1, 16, prefetch=2), 3, 65)
    assert name == "mg::k_smooth3d<double, 0, false, 16, 2, 4, 8>" and needed == 24 * 63**3
    assert profsum.norm_launch(info("sweep", 1, 32, waves=4), 2, 129)[0] == "mg::k_smooth2d<double, 0, false, 32, 4>"


def test_sweeps_by_colour_keep_their_name():
    raw = "void mg::(anonymous namespace)::k_smooth3d_rb<float, 0, 8, 2>(mg::GridDesc const*, int, int)"
    assert profsum.short_name(raw) == "mg::k_smooth3d_rb<float, 0, 8, 2>"
    assert profsum.launched_sweep(3, 4, 8, 1, wv=1, flags=2) == "mg::k_smooth3d_rb<float, 0, 8, 2>"
    # rows with coefficients, and every sweep with more wavefronts
    assert profsum.launched_sweep(3, 4, 8, 2, True, 1) == profsum.sweep_kernel(3, 4, 8, 2, True, 1)
    assert profsum.launched_sweep(3, 8, 16, 2, wv=8) == profsum.sweep_kernel(3, 8, 16, 2, wv=8)


def test_traffic_by_kernel_and_grid(tmp_path):
    """Two counter runs: finest-level launches by name and workgroups, calibrated on the copy, idle ones left out."""
    sweep = "void mg::(anonymous namespace)::k_smooth3d_x2<float, 0, 2, 8, 2>(mg::GridDesc const*, int, int)"
    copy = "void mg::(anonymous namespace)::k_copy_bytes(uint4*, uint4 const*, unsigned long)"
    for cname, kib, unit in (("FETCH_SIZE", 500000.0, 2.0), ("WRITE_SIZE", 400000.0, 1.0)):
        con = sqlite3.connect(tmp_path / f"{cname}.db")
        con.execute("create table counters_collection (kernel_name text, grid_size_x int, workgroup_size_x int, "
                    "counter_name text, value real)")
        rows = [(copy, 256, 256, 1048576.0 / unit), (sweep, 512 * 7, 512, kib), (sweep, 512 * 7, 512, kib),
                (sweep, 512 * 7, 512, 1.0), (sweep, 512, 512, 10.0)]  # stop flag set; a coarse level
        con.executemany(f"insert into counters_collection values (?, ?, ?, '{cname}', ?)", rows)
        con.commit()
        con.close()
    (tmp_path / "bench.json").write_text(json.dumps(
        {"config": {"dim": 3, "n": 513, "workload": "poisson3d_513_fp32ir"}, "dtype": "f32+f64"}) + "\n")
    rec = profsum.traffic(str(tmp_path / "FETCH_SIZE.db"), str(tmp_path / "WRITE_SIZE.db"), str(tmp_path / "bench.json"))
    (e,) = rec["launches"]
    assert (e["kernel"], e["blocks"]) == ("mg::k_smooth3d_x2<float, 0, 2, 8, 2>", 7)
    assert e["bytes_per_launch"] == pytest.approx(1024 * (2.0 * 500000.0 + 400000.0))
    assert e["read"] == pytest.approx(1024 * 2.0 * 500000.0) and e["dispatches"] == 2
