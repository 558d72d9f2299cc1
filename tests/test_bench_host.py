"""Host-side helpers of bench.py (no GPU): the oracle process pool returns results in
order and is closed and joined (not terminated), the baseline states both the
processes it used and the host's cores, and the traffic summary adds up one call."""
import os

import bench


def _square(x):
    return x * x


def test_pool_map_returns_results_in_order():
    assert bench.pool_map(_square, list(range(20)), 3) == [x * x for x in range(20)]


def test_oracle_pool_size_and_core_fields():
    host = len(os.sched_getaffinity(0))
    p = bench.oracle_procs()
    assert 1 <= p <= min(host, bench.BOX_CPU_SHARE)
    assert bench.oracle_procs(2) <= 2
    f = bench.cores_fields(p)
    assert f["cores"] == p and f["host_cores"] == host and str(host) in f["cores_note"]


def test_traffic_summary_adds_up_a_call(tmp_path, capsys):
    """Two calls, each one launch of a<1, true> and three of b: KiB per call, scaled by the copy kernel."""
    def runs(sub, counter, rows):
        (tmp_path / sub).mkdir()
        with open(tmp_path / sub / "run_counter_collection.csv", "w") as f:
            f.write("Kernel_Name,Counter_Name,Counter_Value\n")
            f.writelines(f'"{k}",{counter},{v}\n' for k, v in rows)

    kib = bench.COPY_WORDS * 4 / 1024
    for sub, counter, copy in (("fetch", "FETCH_SIZE", kib / 2), ("write", "WRITE_SIZE", kib)):
        runs(f"copy_{sub}", counter, [("void at::neg_kernel(int)", copy)] * 5)
        runs(sub, counter, [("void ckks::(anonymous namespace)::a<1, true>(int)", 7.0)] * 2
             + [("ckks::(anonymous namespace)::b(int)", 10.0)] * 6)
    bench.summarize_traffic(str(tmp_path), ("a<1, true>", "b"), bench.RNS_SOURCE)
    out = capsys.readouterr().out
    assert f"fetch_bytes_per_launch: {37 * 1024 * 2:.6g}" in out and f"write_bytes_per_launch: {37 * 1024:.6g}" in out
    assert "per call (3 launches)" in out
