"""Which plans march from segment tables, and that their 32-bit offsets hold
every place they reach (host code, on a stand-in for the HIP runtime)."""
import pytest

from host_runtime import run


@pytest.mark.parametrize("nx,nz", [
    (4096, 4096),   # offsets up to 2^24 - 1 cells
    (4095, 4097),   # cascade 6: a probe in row 4128 reaches row 0, 4128 x 4095 > 2^24 cells
    (65280, 257),
    (257, 65280),
    (4000, 4000),
])
def test_segment_keys_hold_every_offset(tmp_path, nx, nz):
    """A segment's key is the byte offset, at 128 B a cell, from its probe's
    cell to the cell crossed, in 32 bits with sign. Probes of a ragged grid
    lie past its far edge, so the offset can pass 2^24 cells on a grid that
    holds fewer: such plans walk, the others keep their tables."""
    far = 0
    for i in range(10):
        s = 1 << i
        if i and 1.5 * 4 ** (i - 1) >= ((nx + s) ** 2 + (nz + s) ** 2) ** 0.5:
            continue  # every ray starts outside the domain
        x0 = (-(-nx // s) - 1) * s + s // 2
        z0 = (-(-nz // s) - 1) * s + s // 2
        far = max(far, max(z0, nz - 1) * nx + max(x0, nx - 1))
    tables = far * 128 < 2**31
    assert tables == ((nx, nz) in [(4096, 4096), (257, 65280), (4000, 4000)])
    run(tmp_path, f"""
        p = plan({nx}, {nz})
        built = count(launches(), "k_build_tables")
        ls = solve(p, {nx}, {nz})
        assert (built > 0) == {tables}, built
        assert (count(ls, "k_march_table") > 0) == {tables}
        assert (count(ls, "k_march_rows") > 0) == (not {tables})
    """)


@pytest.mark.parametrize("nx,nz,n_cascades,f16", [
    (8, 140000, 10, False), (8, 140000, 10, True), (8, 131072, 10, True), (8, 120000, 10, True), (333, 200, 0, True)])
def test_cascade_places_fit_32_bits(tmp_path, nx, nz, n_cascades, f16):
    """The march's places in a stored cascade (16 wavelengths of every
    direction's 16-bit code, or of the FP32 means of 4) are 32-bit: a plan with
    a cascade of more walks. On 8 x 140000 the cascade of spacing 512 holds 274
    probes x 2^20 directions."""
    n = n_cascades or 7
    most = max(-(-nx // 2**i) * -(-nz // 2**i) * 4 ** (i + 1) * 16 // (1 if f16 else 4) for i in range(1, n))
    tables = most < 2**32
    assert tables == ((nx, nz, f16) not in [(8, 140000, True), (8, 131072, True)])
    run(tmp_path, f"""
        p = plan({nx}, {nz}, storage={int(f16)}, n_cascades={n_cascades})
        assert (count(launches(), "k_build_tables") > 0) == {tables}
        ls = solve(p, {nx}, {nz})
        assert (count(ls, "k_march_table") > 0) == {tables}
        assert (count(ls, "k_march_rows") > 0) == (not {tables})
    """)


@pytest.mark.parametrize("nx,nz,windowed,most", [(512, 512, 1, 2**17), (64, 140000, 1, 2**27), (1500, 1500, 2, 2**20)])
def test_window_bins_follow_the_lists(tmp_path, nx, nz, windowed, most):
    """The bins that sort a windowed cascade's workgroups by (window, region,
    wedge) are as many as its longest list has windows (the cascade of spacing
    16 on 512^2: 288 cells x sqrt 2, so 4 windows of 128, on 8 x 8 regions in
    32 wedges), 2^25 at most."""
    run(tmp_path, f"""
        p = plan({nx}, {nz})
        n = count(launches(), "k_windows") // 2
        assert n >= {windowed}, n
        bins = mallocs()[2:2 + 2 * n:2]
        assert all(b <= {most} for b in bins), bins
    """)


@pytest.mark.parametrize("t1", [1e306, 1e308, 1.7e308])
def test_intervals_near_the_largest_double(tmp_path, t1):
    """With the bilinear fix the end of an interval overflows; such lists are
    not sized from infinities, the plan walks."""
    run(tmp_path, f"""
        p = plan(64, 64, flags=1, c0_t1={t1})
        assert all(b < 2**31 for b in mallocs())
        ls = solve(p, 64, 64)
        if count(ls, "k_march_fix_table") == 0:
            assert count(ls, "k_march_fix") > 0
    """)


def test_headers_of_lists_that_are_too_many(tmp_path):
    """A plan whose lists cannot fit makes no host copy of their headers: 12
    cascades on 8^2 have 2^24 directions, 0.7 GB of them on host and (here)
    device each, 1.1 GB of headers."""
    run(tmp_path, """
        p = plan(8, 8, n_cascades=12, c0_t1=1e-6)
        assert count(launches(), "k_build_tables") == 0
        peak = [int(l.split()[1]) for l in open("/proc/self/status") if l.startswith("VmHWM")][0]
        assert peak < 2_000_000, peak
    """)
