"""The new half of a 512-row buffer kept in pieces of bf16: every way rows reach it and every reader of it must agree with the
same stream kept as fp32 (all-parts arithmetic, same bits) or with plain fp32 rows."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _rows(n, D, seed):
    import torch

    g = torch.Generator(device="cuda").manual_seed(seed)
    U = torch.randn(n, 40, generator=g, device="cuda") * torch.arange(1, 41, device="cuda") ** -0.5
    return (U @ torch.randn(40, D, generator=g, device="cuda") + 0.05 * torch.randn(n, D, generator=g, device="cuda")).to(torch.bfloat16)


# widths: whole pieces, ragged, odd; a sketch that fills the half and one that does not; batches that leave the half part full
@pytest.mark.parametrize("D", [640, 1000, 2051])
@pytest.mark.parametrize("ell", [200, 256])
def test_same_bits_as_with_all_parts(D, ell):
    import torch

    from paper_2510_02470_amd.binding import Sage

    G = _rows(4 * ell + 77, D, D + ell)
    out = []
    for mode in (1, 2):
        s = Sage(ell, D, dtype="bf16")
        s.set_update_arithmetic(mode)
        for lo in range(0, G.shape[0], 97):
            s.fd_update(G[lo:lo + 97].contiguous())
        s.fd_update(G[:3 * ell].contiguous())          # looks ahead
        s.fd_basis(100)                                # part of the new half in use
        out.append((s.basis(), s.sketch(), s.stats()))
        s.close()
    assert torch.equal(out[0][0], out[1][0]) and torch.equal(out[0][1], out[1][1])
    assert out[0][2].frob2 == out[1][2].frob2


# The kernel that stores rows and forms their Gram block (four slabs of 16 columns at a time): rows that end within a slab, with one, in
# the middle of a stage and with it; one, several and no whole stages a work-group; rows on any element. All parts: two kernels.
@pytest.mark.parametrize("ell,D,shift", [(129, 257, 0), (256, 320, 1), (256, 336, 0), (200, 14_400, 0), (256, 14_401, 1), (256, 28_672, 0),
                                         (131, 57_391, 1), (256, 57_344, 0)])
def test_same_bits_where_rows_are_stored_and_multiplied_in_one_go(ell, D, shift):
    import torch

    from paper_2510_02470_amd.binding import Sage

    n = 4 * ell + 5
    mem = torch.empty(n * D + 8, dtype=torch.bfloat16, device="cuda")
    G = mem[shift:shift + n * D].view(n, D)
    G.copy_(_rows(n, D, D + ell))
    out = []
    for mode in (1, 2):
        s = Sage(ell, D, dtype="bf16")
        s.set_update_arithmetic(mode)
        s.fd_update(G)
        out.append((s.sketch(), s.stats()))
        s.close()
    assert torch.equal(out[0][0], out[1][0])
    assert out[0][1].frob2 == out[1][1].frob2 and out[0][1].sum_delta == out[1][1].sum_delta


def test_fp32_rows_and_readers_in_the_middle_of_a_half():
    import torch

    from paper_2510_02470_amd.binding import Sage

    ell, D = 256, 1003
    G = _rows(3 * ell, D, 1)
    B = _rows(40, D, 2).float() * 1.0001               # not bf16 values
    a, b = Sage(ell, D, dtype="bf16"), Sage(ell, D, dtype="f32")
    for s, rows in ((a, G), (b, G.float())):
        s.fd_update(rows[:ell + 100].contiguous())     # 100 rows in the new half
        e1 = s.stats().frob2
        s.fd_merge(B)                                  # widens it
        s.fd_update(rows[ell + 100:2 * ell].contiguous())
        if s is a:
            s.set_update_arithmetic(0)                 # fp32 from here: widens what is in pieces
            s.set_update_arithmetic(1)
        s.fd_update(rows[2 * ell:].contiguous())
        s.e = (e1, s.stats().frob2, s.sketch())
    scale = b.e[2].abs().max()
    assert abs(a.e[0] - b.e[0]) <= 1e-6 * b.e[0] and abs(a.e[1] - b.e[1]) <= 1e-6 * b.e[1]
    Ga, Gb = a.e[2].double(), b.e[2].double()
    assert (Ga.T @ Ga - Gb.T @ Gb).norm() <= 1e-5 * (Gb.T @ Gb).norm() and scale > 0
    assert np.isfinite(a.e[1])
