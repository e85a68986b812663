"""bench.py's byte model of the products with B taken in one pass: B once, the
column sums written by the pass and read by the launch that adds them up."""
import bench
import sdpgen


def test_one_pass_bytes():
    inst = sdpgen.workload_banded()
    m, nnz, part = inst.m, inst.nnz, 8 * 16 * inst.nnz
    two = bench.stage_bytes_flops([inst], "fp32", 1.0)
    one = bench.stage_bytes_flops([inst], "fp32", 1.0, part_bytes=part)
    assert one["A_v"]["bytes"] == 8 * m * nnz + 8 * nnz + 16 * m + part
    assert one["AT_y"]["bytes"] == part + 24 * nnz
    assert one["scatter"] == two["scatter"] and "Linv_r" not in one and "LinvT_y" not in one
    tri = 8 * m * (m + 1) // 2 + 16 * m
    h = bench.stage_bytes_flops([inst], "fp32", 1.0, "hsde", part_bytes=part)
    assert h["A_v"]["bytes"] == one["A_v"]["bytes"] + tri and h["LinvT_y"]["bytes"] == tri
    assert "Linv_r" not in h and h["AT_y"] == one["AT_y"]


def test_sparse_instances_beside():
    """Sparse instances of the handle keep their own passes."""
    dense = sdpgen.block_arrow_instance(6, 9, 4, 40, seed=2)
    sparse = sdpgen.block_arrow_instance(6, 9, 4, 40, seed=2, density=0.2)
    both = bench.stage_bytes_flops([dense, sparse], "fp32", 1.0, part_bytes=800)
    d = bench.stage_bytes_flops([dense], "fp32", 1.0, part_bytes=800)
    s = bench.stage_bytes_flops([sparse], "fp32", 1.0)
    for k in ("A_v", "AT_y"):
        assert both[k]["bytes"] == d[k]["bytes"] + s[k]["bytes"]


def test_roofline_takes_the_sums():
    inst = sdpgen.workload_banded()
    r = bench.roofline_of([inst], {"A_v": 0.048, "AT_y": 0.003, "projection": 0.013}, 1.0, "primal",
                          {}, "no_such_workload", 4080640)
    assert r["algorithmic_bytes_per_launch"] == 8 * inst.m * inst.nnz + 8 * inst.nnz + 16 * inst.m + 4080640
