"""Launches whose grids would pass the runtime's 2^32 work items along an axis
are split (host code, on a stand-in for the HIP runtime that refuses them)."""
from host_runtime import run


def test_march_of_a_long_strip(tmp_path):
    """8 x 262144: the cascade of spacing 512 has 512 probes x 2^20 directions,
    2^24 workgroups of 4 directions x 8 probes."""
    run(tmp_path, """
        p = plan(8, 262144, n_wave=16, n_cascades=10, c0_t1=2.0)
        assert count(launches(), "k_build_tables") > 0
        n = 512 // 8 * 2**18
        big = [l for l in solve(p, 8, 262144, 16) if "k_march_table" in l[0]]
        assert sum(l[1] for l in big[:2]) == n and big[0][1] < 2**24, big[:3]
        assert len(big) == 11
    """)


def test_march_beside_a_narrow_last_batch(tmp_path):
    """The same with 17 wavelengths: every launch is within the limits."""
    run(tmp_path, """
        p = plan(8, 262144, n_wave=17, n_cascades=10, c0_t1=2.0)
        solve(p, 8, 262144, 17)
    """)


def test_emergent_beam(tmp_path):
    """A beam of 8 million rays across 4096^2 cells: 256 pieces x 2^17 groups."""
    run(tmp_path, """
        nx = nz = 4096
        p = plan(nx, nz)
        n = 8 << 20
        f, I = device(4 * nx * nz), device(4 * n)
        launches()
        rc = L.rcx_emergent(p, 1, f, f, 1.0, 0.1, n, I, None)
        assert rc == 0, rc
        ls = launches()
        groups = [l[1] // 256 for l in ls if "k_emergentILb" in l[0]]
        assert sum(groups) == n // 64 and len(groups) > 1, ls
    """)


def test_batch_of_many(tmp_path):
    """300 atmospheres of 256^2 x 128 wavelengths: 2e7 workgroups a cascade."""
    run(tmp_path, """
        n, nx, nw = 300, 256, 128
        L.rcx_batch_create.argtypes = [C.c_int32, C.POINTER(rcx.rcx_grid), C.POINTER(C.c_int32),
                                       C.POINTER(rcx.rcx_params), C.POINTER(C.c_void_p)]
        b = C.c_void_p()
        assert L.rcx_batch_create(n, (rcx.rcx_grid * n)(*[rcx.rcx_grid(nx, nx, 1.0)] * n), (C.c_int32 * n)(*[nw] * n),
                                  C.byref(params()), C.byref(b)) == 0
        assert L.rcx_batch_set_graph(b, 0) == 0
        f = device(4 * nx * nx * nw)
        arr = (C.c_void_p * n)(*[f] * n)
        launches()
        rc = L.rcx_batch_solve(b, arr, arr, arr, None)
        assert rc == 0, rc
        ls = [l for l in launches() if "k_march_tasks" in l[0]]
        # cascades 1 to 4 (the rays of the top one miss the domain), and
        # cascade 0, 16 probes of a cone a workgroup, in one launch
        per = n * nw // 16 * (nx * nx * 4 // 32)
        assert len(ls) == 2 * 4 + 1 and sum(l[1] for l in ls) == 4 * per + per // 2, (len(ls), per, ls[:4])
    """)
