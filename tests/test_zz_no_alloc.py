"""The allocation-free Pauli-Villars products (dwf_pv_apply_noalloc) against
dwf_pv_apply and the oracle, through the C ABI.

Each mode is called twice in a row on the static scratch array, the second
time with a smaller input, so that stale contents of the first call sit beyond
the second call's field: the results must still equal dwf_pv_apply's bit for
bit (both run the same stencil kernels) and the FP64 oracle to 1e-13."""
import numpy as np
import pytest
import torch

from oracle import dwf_oracle as O
from paper_2004_07732_amd import inputs

pytestmark = pytest.mark.gpu

dwfmg = pytest.importorskip("paper_2004_07732_amd.dwfmg")
DEV = "cuda"

MODES = ["DWF_PV", "DWF_PV_DAG", "DWF_PVDAG_DW", "DWF_PVDAG_DW_DAG"]


def oracle_mode(mode, U, psi, m, M5):
    if mode == "DWF_PV":
        return O.pv(U, psi, M5)
    if mode == "DWF_PV_DAG":
        return O.pv(U, psi, M5, dagger=True)
    if mode == "DWF_PVDAG_DW":
        return O.pv_dag_dw(U, psi, m, M5)
    return O.pv_dag_dw_dagger(U, psi, m, M5)


# (Lx, Ly, Ls, nrhs): a large call, then a smaller one with a ragged lattice
CALLS = [(64, 32, 8, 3), (24, 20, 6, 1)]


@pytest.mark.parametrize("mode", MODES)
@pytest.mark.parametrize("dtype", [torch.complex128, torch.complex64])
def test_noalloc_matches_pv_apply_on_two_calls(mode, dtype):
    m, M5 = 0.03, -1.05
    code = getattr(dwfmg, mode)
    for k, (Lx, Ly, Ls, nrhs) in enumerate(CALLS):
        print(f"noalloc {mode} {dtype} call {k}: {Lx}x{Ly}x{Ls} x {nrhs}", flush=True)
        U = inputs.metropolis_u1(Lx, Ly, 6.0, 10, 500 + k).U
        psi = inputs.gaussian_field((nrhs, Ls, Ly, Lx, 2), 510 + k)
        Ut = torch.from_numpy(U).to(DEV).to(dtype)
        pt = torch.from_numpy(psi).to(DEV).to(dtype)
        got = dwfmg.dwf_pv_apply_noalloc(Ut, pt, m, M5, code)
        want = dwfmg.dwf_pv_apply(Ut, pt, m, M5, code)
        torch.cuda.synchronize()
        assert torch.equal(got, want), f"call {k}: differs from dwf_pv_apply"
        if dtype == torch.complex128:
            ref = oracle_mode(mode, U, psi, m, M5)
            err = np.linalg.norm(got.cpu().numpy() - ref) / np.linalg.norm(ref)
            assert err < 1e-13, f"call {k}: oracle error {err}"


def test_noalloc_rejects_what_does_not_fit():
    """A product whose intermediate field exceeds the static array returns
    DWF_ESCRATCH; the exact-inverse mode is not offered; the single-stencil
    modes have no intermediate field and take any size."""
    cap = dwfmg.noalloc_max_bytes()
    assert cap == 64 << 20
    Lx = Ly = 128
    Ls = 16
    nrhs = cap // (16 * 2 * Lx * Ly * Ls) + 1        # one rhs more than fits in FP64
    U = torch.ones((2, Ly, Lx), dtype=torch.complex128, device=DEV)
    psi = torch.zeros((nrhs, Ls, Ly, Lx, 2), dtype=torch.complex128, device=DEV)
    with pytest.raises(dwfmg.DwfError) as e:
        dwfmg.dwf_pv_apply_noalloc(U, psi, 0.01, -1.0, dwfmg.DWF_PVDAG_DW)
    assert e.value.code == dwfmg.DWF_ESCRATCH
    with pytest.raises(dwfmg.DwfError) as e:
        dwfmg.dwf_pv_apply_noalloc(U, psi[:1], 0.01, -1.0, dwfmg.DWF_PVINV_DW)
    assert e.value.code == dwfmg.DWF_EUNSUPPORTED
    out = dwfmg.dwf_pv_apply_noalloc(U, psi, 0.01, -1.0, dwfmg.DWF_PV)
    torch.cuda.synchronize()
    assert float(out.abs().max()) == 0.0


# no tile divides either: both go through the static array, the first to well beyond the second's field
RAGGED_CALLS = [(60, 36, 8, 3), (24, 20, 6, 1)]


@pytest.mark.parametrize("mode", MODES)
@pytest.mark.parametrize("dtype", [torch.complex128, torch.complex64])
def test_noalloc_on_a_used_array(mode, dtype):
    m, M5 = 0.03, -1.05
    code = getattr(dwfmg, mode)
    bar = 1e-13 if dtype == torch.complex128 else 1e-6   # two stencils of some 30 roundings
    for k, (Lx, Ly, Ls, nrhs) in enumerate(RAGGED_CALLS):
        U = inputs.metropolis_u1(Lx, Ly, 6.0, 10, 520 + k).U
        psi = inputs.gaussian_field((nrhs, Ls, Ly, Lx, 2), 530 + k)
        Ut = torch.from_numpy(U).to(DEV).to(dtype)
        pt = torch.from_numpy(psi).to(DEV).to(dtype)
        got = dwfmg.dwf_pv_apply_noalloc(Ut, pt, m, M5, code)
        assert torch.equal(got, dwfmg.dwf_pv_apply(Ut, pt, m, M5, code)), f"call {k}: differs from dwf_pv_apply"
        ref = oracle_mode(mode, Ut.to(torch.complex128).cpu().numpy(), pt.to(torch.complex128).cpu().numpy(), m, M5)
        assert np.linalg.norm(got.cpu().numpy() - ref) < bar * np.linalg.norm(ref)
