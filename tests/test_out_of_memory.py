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


def test_workspace_without_memory(tmp_path):
    """Where the workspace finds no memory beside the tables, the plan gives
    its tables up and walks; nothing is left behind when the plan is freed."""
    run(tmp_path, """
        before = rt.fake_live_bytes()
        p = plan(512, 512, 16)
        n_windowed = count(launches(), "k_windows") // 2
        assert L.rcx_plan_destroy(p) == 0 and rt.fake_live_bytes() == before
        ws = 2 + 2 * n_windowed  # directions, tables, {bins, lists} of each windowed cascade, workspace
        for refused, tables in ((1, True), (2, False)):
            rt.fake_fail_malloc(ws, refused)
            p = plan(512, 512, 16)
            rt.fake_fail_malloc(0, 0)
            ls = solve(p, 512, 512, 16)
            assert (count(ls, "k_march_table") > 0) == tables and (count(ls, "k_march_rows") > 0) != tables, ls
            n = C.c_size_t()
            assert L.rcx_plan_workspace_bytes(p, 16, C.byref(n)) == 0
            f = device(4 * 16 * 512 * 512)
            assert L.rcx_formal_solve(p, 16, f, f, f, device(n.value), n.value, None) == 0
            L.rcx_plan_destroy(p)
        before = rt.fake_live_bytes()
        for nth, code in ((0, rcx.RCX_E_HIP), (ws, rcx.RCX_E_NOMEM)):
            rt.fake_fail_malloc(nth, 1000)
            try:
                plan(512, 512, 16)
                assert False
            except rcx.RcxError as e:
                assert e.code == code and "hipMalloc" in str(e), e
            rt.fake_fail_malloc(0, 0)
            assert rt.fake_live_bytes() == before
    """)


def test_solver_without_memory(tmp_path):
    """The non-LTE solver: where one of its buffers finds no memory beside its
    plan's tables, it is made without them."""
    run(tmp_path, """
        from paper_2408_14425_amd import workloads
        atm = workloads.nlte_atmosphere(64, seed=5, n_line=16, n_cont=8)
        def create():
            return rcx.rcx_nlte_create(rcx.rcx_grid(64, 64, 1.0), params(), rcx.atom_from_dict(atm.atom), atm.lambda_nm,
                                       atm.trans, atm.dnu)
        before = rt.fake_live_bytes()
        h = create()
        assert count(launches(), "k_build_tables") > 0
        full = rt.fake_live_bytes()
        rcx.rcx_nlte_destroy(h)
        assert rt.fake_live_bytes() == before
        rt.fake_fail_malloc(12, 1)  # (a buffer of the solver)
        h = create()
        rt.fake_fail_malloc(0, 0)
        assert count(launches(), "k_build_tables") > 0 and rt.fake_live_bytes() < full
        rcx.rcx_nlte_destroy(h)
        assert rt.fake_live_bytes() == before
    """)
