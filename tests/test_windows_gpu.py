"""Cascades marched in windows (march_table.hip) where several things meet: more
than one whole batch (one batch's ray state at a time) with 16-bit cascades,
with flagged probes and beside a narrower last batch; a widest cascade of 16
directions; and the non-LTE solver's continuum, whose state lies in a buffer of
its own (line groups of fewer than 4 batches) or in the cascades' free slots.
Formal solves equal, bit for bit, their batches solved one by one in a workspace
that holds no state (every cascade marched whole); the continuum's J is held to
the FP64 oracle at the parity bars (1e-4; 1e-3 with 16-bit cascades)."""
import numpy as np
import pytest

from host_runtime import run
from paper_2408_14425_amd import workloads as W

SOLVES = [
    # nx, nz, wavelengths, plan options, flagged share
    (330, 300, 33, {}, None),
    (330, 300, 40, {"storage": 1}, None),
    (340, 300, 33, {}, 0.03),
    (340, 300, 34, {"storage": 1}, 0.2),
    (400, 400, 16, {"c0_t1": 150.0, "n_cascades": 3}, None),
    (260, 600, 32, {}, 0.4),
    (350, 340, 32, {"bilinear_fix": True}, None),
]
NLTE = [
    # wavelengths per line (2 lines), storage, share of the cells flagged
    (20, 0, None),   # two batches a line: the state's own buffer
    (20, 1, None),
    (20, 0, 0.3),
    (64, 1, None),   # four: in slots 2 and 3 of a cascade buffer
    (64, 1, 0.3),
]
NX, NZ = 330, 300


def test_these_grids_have_windows(tmp_path):
    for nx, nz, n_wave, opts, _ in SOLVES:
        kw = {("flags" if k == "bilinear_fix" else k): (1 if k == "bilinear_fix" else v) for k, v in opts.items()}
        run(tmp_path, f"""
            plan({nx}, {nz}, {n_wave}, **{kw!r})
            assert count(launches(), "k_windows") > 0
        """)


def _torch():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch


@pytest.mark.gpu
@pytest.mark.parametrize("nx,nz,n_wave,opts,flagged", SOLVES)
def test_windows_equal_whole_marches(nx, nz, n_wave, opts, flagged):
    torch = _torch()
    from paper_2408_14425_amd import rcx
    inp = W.line_medium(nx, n_wave, seed=7, nz=nz)
    print(f"[gpu] windows {nx}x{nz} w{n_wave} {opts} flagged {flagged}", flush=True)
    plan = rcx.Plan(nx, nz, n_wave, **opts)
    if flagged:
        plan.set_active(W.active_cells(nx, nz, seed=4, frac=flagged))
    chi, eta = torch.from_numpy(inp.chi).cuda(), torch.from_numpy(inp.eta).cuda()
    J = plan.formal_solve(chi, eta, torch.full_like(chi, float("nan")))
    parts = []
    for lo in range(0, n_wave, 16):
        c, e = chi[lo:lo + 16].contiguous(), eta[lo:lo + 16].contiguous()
        ws = None
        if len(c) >= 8 and not opts.get("bilinear_fix"):
            # between the need without the state and that with it (64 B an
            # entry of the largest cascade more); the fix sums its taps in
            # another order there, so its batches keep their windows
            most = max(plan.work().level_rays)
            ws = torch.empty(plan.workspace_bytes(len(c)) - 32 * most, dtype=torch.uint8, device="cuda")
        parts.append(plan.formal_solve(c, e, workspace=ws))
    torch.cuda.synchronize()
    plan.close()
    assert torch.equal(J, torch.cat(parts))
    assert (J > 0).any()


@pytest.mark.gpu
@pytest.mark.parametrize("n_line,storage,flagged", NLTE)
def test_continuum_windows_match_oracle(n_line, storage, flagged):
    torch = _torch()
    from oracle import nlte
    from paper_2408_14425_amd import rcx
    inp = W.nlte_atmosphere(NX, seed=6, n_line=n_line, n_cont=20, nz=NZ)
    t_cut = float(np.quantile(inp.T, flagged)) if flagged else None
    print(f"[gpu] continuum windows {n_line} {storage} {flagged}", flush=True)
    s = rcx.Nlte(inp, storage=storage)
    if flagged:
        s.set_temperature_cut(t_cut)
    _, J = s.formal_solve_rates(s.lte(), want_J=True)
    torch.cuda.synchronize()
    Jg = J.cpu().numpy().reshape(inp.n_wave, -1).astype(np.float64)
    s.close()
    P = nlte.Problem(inp, t_cut=t_cut)
    lams = np.array([n_line // 2, 2 * n_line, 2 * n_line + 15, 2 * n_line + 19])  # a line, and both continuum batches
    Jo = P.formal_solve(P.lte, lams=lams)[0]
    on = slice(None) if t_cut is None else P.T < t_cut
    rel = np.abs(Jg[lams][:, on] - Jo[:, on]) / Jo[:, on]
    print(f"J max rel {rel.max(axis=1)}")
    if flagged:
        assert not Jg[:, ~on].any()
    assert rel.max() < (1e-3 if storage else 1e-4)
