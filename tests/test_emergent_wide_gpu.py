"""An emergent beam of 2^31 - 1 rays (rcx_emergent's largest): its last groups
of 64 reach past the largest 32-bit index. The rays that cross the grid equal
those of a narrow beam, the others are dark."""
import pytest

pytestmark = pytest.mark.gpu


def test_the_widest_beam():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2408_14425_amd import rcx
    nx, nz, n = 64, 16, 2**31 - 1
    print("[gpu] widest beam", flush=True)
    plan = rcx.Plan(nx, nz, 1)
    g = torch.Generator(device="cuda").manual_seed(2)
    chi = torch.rand((1, nz, nx), device="cuda", generator=g) * 0.1 + 0.01
    eta = torch.rand((1, nz, nx), device="cuda", generator=g)
    narrow = plan.emergent(chi, eta, 0.6, 0.8, 255)
    wide = torch.full((1, n), float("nan"), device="cuda")
    plan.emergent(chi, eta, 0.6, 0.8, n, I=wide)
    torch.cuda.synchronize()
    plan.close()
    lo = (n - 255) // 2
    assert torch.equal(wide[:, lo:lo + 255], narrow)
    assert (narrow > 0).sum() > 40
    # (a NaN counts; in pieces, for the memory of the comparison)
    lit = sum(int((wide[0, a:a + (1 << 28)] != 0).sum()) for a in range(0, n, 1 << 28))
    assert lit == int((narrow != 0).sum())
