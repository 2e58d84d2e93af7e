"""The coarse operator of 16 and more components on the vector units (FP64 and FP32 links, and
16-bit links whose n is no multiple of 16) at the edges of its column tiles, against the oracle."""
import numpy as np
import pytest
import torch

from oracle import dwf_oracle as O
from paper_2004_07732_amd import inputs

pytestmark = pytest.mark.gpu

dwfmg = pytest.importorskip("paper_2004_07732_amd.dwfmg")
M, M5 = 0.05, -1.0


def T(x):
    return torch.from_numpy(np.ascontiguousarray(x)).to("cuda")


def pair(Lx, Ly, nvec, block, Lsc, ncol, link, seed):
    U = inputs.metropolis_u1(Lx, Ly, 6.0, 20, seed).U
    start = inputs.gaussian_field((nvec, Ly, Lx, 2), seed + 1)
    p = dwfmg.MGParams(nvec=[nvec], block=[block], Ls_coarse=[Lsc], link_prec=[link], vec_prec=[dwfmg.P_F64],
                       setup_iters=0)
    mg = dwfmg.MG(T(U), 4, M, M5, p, [T(start)], max_nrhs=ncol)
    o = O.MG(U, 4, M, M5, O.MGParams(levels=[O.LevelParams(nvec=nvec, block=block[::-1], Ls=Lsc, setup_iters=0)]),
             [start])
    return mg, o


def check(mg, o, S, shape, bar, seed):
    x = inputs.gaussian_field(shape, seed)
    ncol = shape[0]
    D = lambda v, m=M, dag=False: O.stencil_dwf(S, v, m, M5, dagger=dag)  # noqa: E731
    for code, want in ((dwfmg.MG_OP_DW, lambda: D(x)), (dwfmg.MG_OP_DW_DAG, lambda: D(x, dag=True)),
                       (dwfmg.MG_OP_A, lambda: D(D(x), 1.0, True))):
        got, w = mg.level_op(1, code, T(x), ncol).cpu().numpy(), want()
        for c in range(ncol):
            assert np.linalg.norm(got[c] - w[c]) < bar * np.linalg.norm(w[c]), (code, c)


@pytest.mark.parametrize("Lsc,ncol", [(2, 1), (3, 1), (2, 2), (5, 1), (4, 2), (3, 3), (2, 9)])
@pytest.mark.parametrize("nvec,block", [(8, (4, 4)), (12, (4, 4)), (16, (4, 4)), (24, (8, 4)), (32, (8, 4))])
def test_column_tiles_fp64(nvec, block, Lsc, ncol):
    """1..18 (right-hand side, slice) columns: tiles of 2, 4 and 8, full and ragged."""
    mg, o = pair(16, 24, nvec, block, Lsc, ncol, dwfmg.P_F64, 940)
    S = o.levels[1].S
    check(mg, o, S, (ncol, Lsc, 24 // block[1], 16 // block[0], 2 * nvec), 1e-13, 941)
    x = inputs.gaussian_field((ncol, 24 // block[1], 16 // block[0], 2 * nvec), 942)
    for code, dag in ((dwfmg.MG_OP_WILSON, False), (dwfmg.MG_OP_WILSON_DAG, True)):
        got = mg.level_op(1, code, T(x), ncol, mass=-0.2).cpu().numpy()
        want = o.levels[1].wilson2d(x, -0.2, dagger=dag)
        assert np.linalg.norm(got - want) < 1e-13 * np.linalg.norm(want)


@pytest.mark.parametrize("Lx,Ly,block", [(4, 4, (4, 4)), (8, 4, (4, 4)), (4, 12, (4, 4))])
def test_coarse_extents_one_two_three(Lx, Ly, block):
    """A site that is its own neighbour, and the same neighbour on both sides."""
    mg, o = pair(Lx, Ly, 8, block, 2, 1, dwfmg.P_F64, 950)
    check(mg, o, o.levels[1].S, (1, 2, Ly // 4, Lx // 4, 16), 1e-13, 951)


def test_tiles_walked_by_one_workgroup():
    """Enough sites that a workgroup takes all column tiles of its site."""
    mg, o = pair(96, 96, 8, (4, 4), 3, 5, dwfmg.P_F64, 960)
    check(mg, o, o.levels[1].S, (5, 3, 24, 24, 16), 1e-13, 961)


@pytest.mark.parametrize("link", ["f32", "bf16", "f16"])
@pytest.mark.parametrize("Lsc,ncol", [(2, 1), (4, 1), (3, 3)])
def test_narrow_links(link, Lsc, ncol):
    """n = 24, links rounded to their storage, FP32 arithmetic: 120 products of unit size
    leave about sqrt(120) x 2^-24 = 6.5e-7; bar 2e-6."""
    lp = {"f32": dwfmg.P_F32, "bf16": dwfmg.P_BF16, "f16": dwfmg.P_F16}[link]
    mg, o = pair(16, 24, 12, (4, 4), Lsc, ncol, lp, 970)

    def rnd(a):
        if link == "f16":   # (rounded once, from FP64)
            return np.asarray(a).astype(np.float16).astype(np.float64)
        f = np.ascontiguousarray(a, dtype=np.float32)
        if link == "f32":
            return f.astype(np.float64)
        u = f.view(np.uint32).astype(np.uint64)
        u = ((u + 0x7FFF + ((u >> 16) & 1)) >> 16) << 16
        return u.astype(np.uint32).view(np.float32).astype(np.float64)

    S = o.levels[1].S
    Sr = O.Stencil(diag=rnd(S.diag.real) + 1j * rnd(S.diag.imag), hop=rnd(S.hop.real) + 1j * rnd(S.hop.imag),
                   chir=S.chir)
    check(mg, o, Sr, (ncol, Lsc, 6, 4, 24), 2e-6, 971)
