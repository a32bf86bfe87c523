"""The cache of rcx_batch_autotune (host code, on a stand-in for the HIP
runtime): a line serves the march, the intervals and the shapes it was tuned on."""
from host_runtime import run


def test_cache_keys(tmp_path):
    run(tmp_path, f"""
        import os
        path = {str(tmp_path / "orders.jsonl")!r}
        # a line of the march before the tables
        open(path, "w").write('{{"v2_f32_64x64w16": 2032, "ms": 1.0}}\\n')
        L.rcx_batch_create.argtypes = [C.c_int32, C.POINTER(rcx.rcx_grid), C.POINTER(C.c_int32),
                                       C.POINTER(rcx.rcx_params), C.POINTER(C.c_void_p)]
        f = device(4 * 16 * 64 * 64)
        arr = (C.c_void_p * 1)(f)
        def tune(**kw):
            b = C.c_void_p()
            assert L.rcx_batch_create(1, C.byref(rcx.rcx_grid(64, 64, 1.0)), (C.c_int32 * 1)(16), C.byref(params(**kw)),
                                      C.byref(b)) == 0
            best = C.c_int32()
            launches()
            assert L.rcx_batch_autotune(b, arr, arr, arr, path.encode(), C.byref(best), None) == 0
            L.rcx_batch_destroy(b)
            return len(launches()) > 0, len(open(path).read().splitlines())
        assert tune() == (True, 2)
        assert tune() == (False, 2)
        assert tune(c0_t1=2.0) == (True, 3)
        assert tune(t_rule=1) == (True, 4)
        assert tune(storage=1) == (True, 5)
        assert tune(c0_t1=2.0) == (False, 5)
    """)
