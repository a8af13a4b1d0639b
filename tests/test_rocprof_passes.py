"""The kernel table of one pass: only what follows the last rest counts, kernels that overlap leave no gap."""
from paper_2607_14025_amd import rocprof_summary as R


def test_passes_after_the_rest(tmp_path):
    f = tmp_path / "t.csv"
    ms = 1000000
    rows = [("k_warm(int)", 0, 5 * ms), ("void stern::k_a<1>(int)", 500 * ms, 502 * ms), ("void stern::k_b(int)", 501 * ms, 503 * ms),
            ("void stern::k_a<1>(int)", 504 * ms, 506 * ms), ("void stern::k_b(int)", 506 * ms, 510 * ms)]
    f.write_text('"Kernel_Name","Start_Timestamp","End_Timestamp"\n' + "".join(f'"{n}",{a},{b}\n' for n, a, b in rows))
    md = R.passes(str(f), "case", 2, 1)
    assert "k_warm" not in md and "k_a" not in md.split("|---|")[1]
    assert "2 launches, 5000.0 us, of which no kernel runs for 500.0 us (10.0%)" in md
    assert "| `k_b` | 1 | 3000.00 | 3000.0 | 60.0% |" in md
