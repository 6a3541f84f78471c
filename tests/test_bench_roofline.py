"""The benchmark's roofline entry names what bounds the kernel that ran (CPU)."""
import pytest

import bench


def _stats(resident, iters, n, launches, ms):
    """The library's counters of `launches` fused launches of n unknowns with
    `iters` CG iterations each."""
    return dict(kernel_launches=launches, kernel_bytes=float(launches * n * (48 * iters + 20)), kernel_ms=ms * launches,
                resident=resident, block=768, cols_per_thread=2, team=3, wave_rows=1)


def test_streaming_form_is_priced_against_memory():
    r = bench.roofline_of(_stats(2, 7, 18_000_000, 100, 1.115), 18_000_000, "no counters")
    assert r["bound"] == "hbm" and r["unit"] == "GB/s" and r["kernel"] == "k_fused_cg<float>"
    assert r["achieved"] == pytest.approx(18e6 * 356 / 1.115e-3 / 1e9) and r["frac"] == r["achieved"] / 8000.0


def test_on_chip_form_is_priced_against_the_vector_units():
    """Its words never reach memory: the method's bytes over its time may pass the
    memory's peak and are no bandwidth."""
    n, iters = 18_000_000, 7
    r = bench.roofline_of(_stats(3, iters, n, 100, 0.5), n, "no counters")
    assert r["bound"] == "valu" and r["unit"] == "TFLOP/s" and r["kernel"] == "k_chip_cg<float>"
    assert r["achieved"] == pytest.approx(bench.CHIP_FLOPS_PER_NODE * n * (iters + 1) / 0.5e-3 / 1e12)
    assert r["frac"] == r["achieved"] / bench.VALU_PEAK_TFLOPS < 1.0
    assert r["method_equivalent_gbs"] > bench.HBM_PEAK_GBS and "no memory traffic" in r["basis"]
    assert r["traffic"] is None and r["measured_dram_frac"] is None
