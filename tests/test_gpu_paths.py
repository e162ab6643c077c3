"""GPU paths chosen by size, at the sizes where they can go wrong, against the oracle.

Amplitudes: 1e-12 (complex128) and 1e-5 (complex64) absolute on normalised states, the bounds of every gate."""
import numpy as np
import pytest
import torch

from oracle import gates as og
from oracle import strings as ost
from paper_2605_03123_amd import synth
from errlog import AMP

pytestmark = pytest.mark.gpu

TOL = {torch.complex128: AMP["complex128"], torch.complex64: AMP["complex64"]}


@pytest.fixture(scope="module")
def ffx():
    assert torch.cuda.is_available(), "GPU tests need a ROCm device"
    from paper_2605_03123_amd import ffx as mod
    return mod


def _state(r, norb, nelec, dtype):
    v = synth.random_state(r, ost.dim(norb, nelec[0]), ost.dim(norb, nelec[1]))
    return torch.from_numpy(v).to(dtype).to("cuda:0")


def _ref(t):
    return t.detach().cpu().to(torch.complex128).numpy()


# one string, a block of 256 strings less one, exactly a few blocks, strings of two lengths, 32 orbitals
@pytest.mark.parametrize("norb,nelec", [(1, (1, 0)), (9, (0, 5)), (10, (5, 1)), (12, (3, 5)), (24, (2, 1)), (32, (1, 2))])
@pytest.mark.parametrize("dtype", [torch.complex128, torch.complex64])
def test_string_tables_of_a_diagonal_gate(ffx, norb, nelec, dtype):
    r = synth.rng([41, norb, nelec[0], nelec[1]])
    v = _state(r, norb, nelec, dtype)
    J = [synth.random_symmetric(r, norb, 0.5) for _ in range(2)]
    Jab = r.normal(0.0, 0.5, (norb, norb))
    lam, lam_b = r.normal(size=norb), r.normal(size=norb)
    out = ffx.apply_diag_coulomb_evolution(v, J[0], 0.7, norb, nelec, J_ab=Jab, J_bb=J[1])
    ffx.apply_num_op_sum_evolution(out, lam, 0.3, norb, nelec, lam_b=lam_b, out=out)
    ref = og.apply_diag_coulomb_evolution(_ref(v), J[0], 0.7, norb, nelec, J_ab=Jab, J_bb=J[1])
    ref = og.apply_num_op_sum_evolution(ref, lam, 0.3, norb, nelec, lam_b=lam_b)
    assert np.max(np.abs(_ref(out) - ref)) <= TOL[dtype]
