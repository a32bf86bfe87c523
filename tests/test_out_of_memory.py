"""What a plan does where the device, or the host, has no memory for its
optional parts (host code, on a stand-in for the HIP runtime)."""
from host_runtime import run


def test_windows_without_memory(tmp_path):
    """A cascade whose window lists find no memory is marched whole: the plan
    is made, and solves."""
    run(tmp_path, """
        p = plan(512, 512, 16)  # directions, tables, then the lists of each windowed cascade
        whole = count(launches(), "k_windows")
        assert whole > 0
        L.rcx_plan_destroy(p)
        for nth in range(2, 2 + whole):
            rt.fake_fail_malloc(nth, 1)
            p = plan(512, 512, 16)
            n = count(launches(), "k_windows")
            assert n < whole, (nth, n)
            rt.fake_fail_malloc(0, 0)
            marched = count(solve(p, 512, 512, 16), "k_march_table")
            assert marched >= 5, marched  # (the stand-in's windows are empty)
            L.rcx_plan_destroy(p)
        # at every later use of the flags, too
        p = plan(512, 512, 16)
        rt.fake_fail_malloc(2, 1000)
        assert L.rcx_plan_set_active_host(p, (C.c_uint8 * (512 * 512))(*[1] * (512 * 512)), None) == 0
        rt.fake_fail_malloc(0, 0)
        assert count(solve(p, 512, 512, 16), "k_mask_j") == 1
        L.rcx_plan_destroy(p)
    """)


def test_flags_without_memory(tmp_path):
    """Flags that find no memory leave the plan dense, its windows too."""
    run(tmp_path, """
        flags = (C.c_uint8 * (512 * 512))(*[1] + [0] * (512 * 512 - 1))
        for nth in (0, 1):
            p = plan(512, 512, 16)
            dense = count(launches(), "k_windows")
            assert L.rcx_plan_set_active_host(p, flags, None) == 0
            rt.fake_fail_malloc(nth, 1)
            launches()
            assert L.rcx_plan_set_active_host(p, flags, None) == rcx.RCX_E_HIP
            rt.fake_fail_malloc(0, 0)
            assert count(launches(), "k_windows") == dense  # the dense windows, not those of the old flags
            assert count(solve(p, 512, 512, 16), "k_mask") == 0
            L.rcx_plan_destroy(p)
    """)
