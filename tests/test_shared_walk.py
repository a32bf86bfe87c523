"""The shared-direction walk of plans without segment tables (march_rows.h,
k_march_shared; rcx_plan_set_order): which launches take it (host code, on a
stand-in for the HIP runtime), and that J is the same bit for bit."""
import pytest

from host_runtime import run


@pytest.mark.parametrize("kw,kernel", [
    ("n_incl=2", "k_march_shared"),
    ("c0_dirs=8", "k_march_shared"),
    ("n_incl=2, storage=1", "k_march_shared"),
    ("n_incl=1", "k_march_table"),
    ("n_incl=2, flags=1", "k_march_fix"),
])
def test_which_plans_share_walks(tmp_path, kw, kernel):
    run(tmp_path, f"""
        p = plan(512, 512, n_wave=32, {kw})
        assert count(solve(p, 512, 512, 32), "k_march_shared") == 0
        assert L.rcx_plan_set_order(p, 4, 4, 32, 128, 1) == 0
        ls = solve(p, 512, 512, 32)
        assert count(ls, {kernel!r}) > 0, ls
        assert (count(ls, "k_march_shared") > 0) == ({kernel!r} == "k_march_shared"), ls
    """)


@pytest.mark.gpu
@pytest.mark.parametrize("nx,nz,n_wave,kw", [
    (64, 64, 16, dict(n_incl=2)), (97, 130, 33, dict(n_incl=3)), (97, 130, 17, dict(n_incl=2, storage=1)),
    (64, 80, 5, dict(c0_dirs=8)),
])
def test_shared_walk_gives_the_same_bits(nx, nz, n_wave, kw):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2408_14425_amd import rcx
    print(f"[gpu] shared walk {nx}x{nz} x {n_wave} {kw}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(4)
    chi = 10.0 ** (2.0 * torch.rand((n_wave, nz, nx), device="cuda", generator=g) - 3.0)
    eta = chi * torch.rand((n_wave, nz, nx), device="cuda", generator=g)
    plan = rcx.Plan(nx, nz, n_wave, **kw)
    J = []
    for shared in (0, 1):
        for i in range(1, plan.work().n_cascades):
            plan.set_order(i, 2 if i == 1 else 4, 16, 32, shared)
        J.append(plan.formal_solve(chi, eta).clone())
    torch.cuda.synchronize()
    plan.close()
    assert torch.equal(J[0], J[1])
