"""rcx_nlte_autotune times the solver's own marches (host code, on a stand-in
for the HIP runtime)."""
from host_runtime import run


def test_times_the_solvers_marches(tmp_path):
    run(tmp_path, f"""
        from paper_2408_14425_amd import workloads
        atm = workloads.nlte_atmosphere(128, seed=5, n_line=64, n_cont=16)
        N = rcx._load_nlte()
        path = {str(tmp_path / "orders.jsonl")!r}.encode()
        for k in range(2):
            h = rcx.rcx_nlte_create(rcx.rcx_grid(128, 128, 1.0), params(), rcx.atom_from_dict(atm.atom), atm.lambda_nm,
                                    atm.trans, atm.dnu)
            launches()
            before = rt.fake_live_bytes()
            assert N.rcx_nlte_autotune(C.c_void_p(h), path, None) == 0
            assert rt.fake_live_bytes() == before
            ls = launches()
            assert (count(ls, "k_march_line") > 0 and count(ls, "k_march_table") > 0) == (k == 0), ls[:3]
            assert count(ls, "k_march_rows") == 0
            rcx.rcx_nlte_destroy(h)
        lines = open(path).read().splitlines()
        assert len(lines) == 1 and "/nlte/l8x4/c1/" in lines[0], lines  # 2 lines x 64 wavelengths, a hit the second time
    """)
