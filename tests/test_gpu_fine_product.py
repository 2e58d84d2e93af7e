"""dwf_pv_apply's products A = D_PV^dag D_DW and A^dag = D_DW^dag D_PV in one launch, on lattices
that each fused tile divides and on one that none does, against the oracle."""
import numpy as np
import pytest
import torch

from oracle import dwf_oracle as O
from paper_2004_07732_amd import inputs

pytestmark = pytest.mark.gpu

dwfmg = pytest.importorskip("paper_2004_07732_amd.dwfmg")


# tiles of 32 x 16, 32 x 8, 16 x 16 and 16 x 8 (FP64 from 32 x 8 on), one tile (its own neighbour),
# none (two launches); both fifth-dimension wraps in one chunk, ragged last chunks
@pytest.mark.parametrize("Lx,Ly", [(32, 16), (64, 48), (32, 24), (48, 32), (16, 16), (16, 24), (16, 8), (20, 12)])
@pytest.mark.parametrize("Ls,nrhs", [(2, 1), (3, 2), (7, 1), (16, 3)])
@pytest.mark.parametrize("dtype", [torch.complex64, torch.complex128])
def test_products_match_the_oracle(Lx, Ly, Ls, nrhs, dtype):
    m, M5 = 0.03, -1.2
    U = inputs.links_from_theta(inputs.random_theta(Lx, Ly, 500 + Lx + Ly))
    x = inputs.gaussian_field((nrhs, Ls, Ly, Lx, 2), 501 + Ls)
    Ut, xt = torch.from_numpy(U).cuda().to(dtype), torch.from_numpy(x).cuda().to(dtype)
    Un, xn = Ut.to(torch.complex128).cpu().numpy(), xt.to(torch.complex128).cpu().numpy()
    # FP32: two stencils of some 30 roundings of 2^-24 each
    bar = 1e-13 if dtype == torch.complex128 else 1e-6
    for mode, m1, m2 in ((dwfmg.DWF_PVDAG_DW, m, 1.0), (dwfmg.DWF_PVDAG_DW_DAG, 1.0, m)):
        got = dwfmg.dwf_pv_apply(Ut, xt, m, M5, mode=mode).cpu().numpy()
        for c in range(nrhs):
            want = O.dwf(Un, O.dwf(Un, xn[c], m1, M5), m2, M5, dagger=True)
            assert np.linalg.norm(got[c] - want) < bar * np.linalg.norm(want), (mode, c)


def test_single_slice_takes_two_launches():
    """Ls = 1: the slice is its own fifth-dimension neighbour."""
    m, M5 = 0.03, -1.0
    U = inputs.links_from_theta(inputs.random_theta(32, 16, 7))
    x = inputs.gaussian_field((2, 1, 16, 32, 2), 8)
    got = dwfmg.dwf_pv_apply(torch.from_numpy(U).cuda(), torch.from_numpy(x).cuda(), m, M5).cpu().numpy()
    for c in range(2):
        want = O.pv_dag_dw(U, x[c], m, M5)
        assert np.linalg.norm(got[c] - want) < 1e-13 * np.linalg.norm(want)


def test_product_allocates_nothing_under_capture():
    """The fused product needs no intermediate field: it can be captured after the scratch is
    released, and every replay gives the eager result."""
    U = torch.from_numpy(inputs.links_from_theta(inputs.random_theta(64, 32, 9))).cuda()
    x = torch.from_numpy(inputs.gaussian_field((1, 4, 32, 64, 2), 10)).cuda()
    want = dwfmg.dwf_pv_apply(U, x, 0.02, -1.0)
    out = torch.empty_like(x)
    dwfmg.release_scratch()
    g, s = torch.cuda.CUDAGraph(), torch.cuda.Stream()
    torch.cuda.synchronize()
    with torch.cuda.graph(g, stream=s):
        dwfmg.dwf_pv_apply(U, x, 0.02, -1.0, out=out)
    for _ in range(3):
        out.zero_()
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, want)


# one slice per workgroup (16 x 8 tiles, then the largest); a whole fifth dimension of three; FP64 in two
# launches; chunks of even length below the longest (FP64: 5 + 4 of 9), and one chunk (FP32)
@pytest.mark.parametrize("Lx,Ly,Ls,nrhs", [(32, 32, 4, 1), (64, 64, 5, 3), (80, 88, 3, 13), (64, 64, 3, 8), (96, 64, 4, 4),
                                           (128, 128, 9, 13)])
@pytest.mark.parametrize("dtype", [torch.complex64, torch.complex128])
def test_products_at_the_lines_of_the_rule(Lx, Ly, Ls, nrhs, dtype):
    """Every choice of tile and chunk against the two stencils one after the other (the same site
    arithmetic up to contraction: a few roundings of each site's some 60 terms) and, in the first
    column, the oracle; then the same under capture, where an intermediate field is not used."""
    m, M5 = 0.04, -1.1
    U = inputs.links_from_theta(inputs.random_theta(Lx, Ly, 510))
    x = inputs.gaussian_field((nrhs, Ls, Ly, Lx, 2), 511)
    Ut, xt = torch.from_numpy(U).cuda().to(dtype), torch.from_numpy(x).cuda().to(dtype)
    bar = 1e-13 if dtype == torch.complex128 else 1e-6
    t = dwfmg.dwf_apply(Ut, xt, m, M5)
    two = dwfmg.dwf_pv_apply(Ut, t, m, M5, mode=dwfmg.DWF_PV_DAG)
    got = dwfmg.dwf_pv_apply(Ut, xt, m, M5)
    assert float((got - two).norm() / two.norm()) < bar
    Un, xn = Ut.to(torch.complex128).cpu().numpy(), xt[0].to(torch.complex128).cpu().numpy()
    want = O.pv_dag_dw(Un, xn, m, M5)
    assert np.linalg.norm(got[0].cpu().numpy() - want) < bar * np.linalg.norm(want)
    out = torch.empty_like(xt)
    dwfmg.release_scratch()
    g, s = torch.cuda.CUDAGraph(), torch.cuda.Stream()
    torch.cuda.synchronize()
    with torch.cuda.graph(g, stream=s):
        dwfmg.dwf_pv_apply(Ut, xt, m, M5, out=out)
    for _ in range(2):
        out.zero_()
        g.replay()
        torch.cuda.synchronize()
        assert float((out - two).norm() / two.norm()) < bar


@pytest.mark.parametrize("noalloc", [False, True])
@pytest.mark.parametrize("shift", [1, -1, 3])
def test_overlapping_output_is_not_raced(noalloc, shift):
    """An output that overlaps the input, a slice or three further: only the one launch would read
    what it has written.  The bits are those of the two stencils one after the other."""
    U = torch.from_numpy(inputs.links_from_theta(inputs.random_theta(64, 64, 12))).cuda()
    Ls, pad = 8, abs(shift)
    x = torch.from_numpy(inputs.gaussian_field((Ls, 64, 64, 2), 13)).cuda()
    apply = dwfmg.dwf_pv_apply_noalloc if noalloc else dwfmg.dwf_pv_apply
    for mode in (dwfmg.DWF_PVDAG_DW, dwfmg.DWF_PVDAG_DW_DAG):
        if mode == dwfmg.DWF_PVDAG_DW:
            want = dwfmg.dwf_pv_apply(U, dwfmg.dwf_apply(U, x, 0.02, -1.0), 0.02, -1.0, dwfmg.DWF_PV_DAG)
        else:
            want = dwfmg.dwf_apply(U, dwfmg.dwf_pv_apply(U, x, 0.02, -1.0, dwfmg.DWF_PV), 0.02, -1.0, dagger=True)
        buf = torch.zeros((Ls + pad, 64, 64, 2), dtype=x.dtype, device="cuda")
        i0, o0 = (0, pad) if shift > 0 else (pad, 0)
        psi, out = buf[i0:i0 + Ls], buf[o0:o0 + Ls]
        psi.copy_(x)
        apply(U, psi, 0.02, -1.0, mode, out=out)
        assert torch.equal(out, want)


def test_pinned_stencil_reaches_the_products():
    """dwf_fine_config governs every operator: a product under a pinned stencil takes the two
    stencils, seen by the intermediate field that it allocates."""
    U = torch.from_numpy(inputs.links_from_theta(inputs.random_theta(128, 128, 14))).cuda()
    x = torch.randn((8, 16, 128, 128, 2), dtype=torch.complex128, device="cuda")   # 64 MB
    out = torch.empty_like(x)
    free = []
    try:
        for pin in (dwfmg.FINE_AUTO, dwfmg.FINE_ROW):
            dwfmg.dwf_fine_config(pin, 4)
            dwfmg.release_scratch()
            dwfmg.dwf_pv_apply(U, x, 0.02, -1.0, out=out)
            torch.cuda.synchronize()
            free.append(torch.cuda.mem_get_info()[0])
            dwfmg.release_scratch()
    finally:
        dwfmg.dwf_fine_config(dwfmg.FINE_AUTO)
    assert free[0] - free[1] >= (48 << 20)
