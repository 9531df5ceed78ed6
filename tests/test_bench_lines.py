"""What the bench line says of kernels: the ceiling on {+,-,*} trees comes from
the counters of the current kernel (its two forms agree, and it is null where
there are none), and a batched step counts all of its launches."""
import bench


def test_unpacked_ceiling_follows_the_counters(monkeypatch):
    ops, launch_s, valu = 3.43e10, 6.0e-4, 2.98e8
    monkeypatch.setattr(bench, "counter_record", lambda workload, kernel: ({"valu_insts": "%d" % valu}, "a file"))
    mix = bench.op_mix_ceiling(ops, launch_s, "kernel", "workload")
    r = {}
    bench.add_unpacked_ceiling(r, mix)
    lane_ops = 256 * 4 * 16 * 2.4e9
    assert abs(r["unpacked_ceiling_tgpops"] * 1e12 / (lane_ops * ops / (64 * valu)) - 1) < 1e-12
    assert abs(r["frac_of_unpacked_ceiling"] / (ops / launch_s / (r["unpacked_ceiling_tgpops"] * 1e12)) - 1) < 1e-12
    assert r["frac_of_unpacked_ceiling"] == mix["frac"]
    assert "performs 1.80 GP operations" in r["unpacked_ceiling_note"]


def test_no_ceiling_without_counters(monkeypatch):
    monkeypatch.setattr(bench, "counter_record", lambda workload, kernel: (None, None))
    r = {}
    bench.add_unpacked_ceiling(r, bench.op_mix_ceiling(1.0, 1.0, "kernel", "workload"))
    assert r["frac_of_unpacked_ceiling"] is None and r["unpacked_ceiling_tgpops"] is None


def test_a_batched_step_counts_all_its_launches():
    ops = 2.3e11
    one = bench.batched_roofline(ops, 20, 700.0, 20, "k_tuned", "w")       # 20 steps of one launch, 35 ms each
    six = bench.batched_roofline(ops, 120, 560.0, 20, "k_tuned", "w")      # six launches a step, 28 ms in all
    assert one["kernel"] == "k_tuned" and abs(one["kernel_ms"] - 35.0) < 1e-9 and "note" not in one
    assert six["kernel"] == "k_core" and abs(six["kernel_ms"] - 28.0) < 1e-9 and six["launches_per_step"] == 6
    assert abs(six["achieved"] - ops / 28e-3 / 1e12) < 1e-9
