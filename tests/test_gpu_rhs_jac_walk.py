"""f and J of more cells than fill the chip at once (the grid walks the cells)
against the same cells in calls that fit (one cell per wave): the same
arithmetic per cell, so equal bit for bit.  5,003 cells are more than two fills
of every size here and leave a ragged end; 17, 32, 33, 55 and 64 components are
the edges of the padded sizes and of the rows of J that one store covers, 11
components never walk."""
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

from paper_2105_12070_amd.inputs import make_mechanism, make_states  # noqa: E402

DEV = "cuda:0"


@pytest.mark.parametrize("K,R", [(10, 24), (16, 40), (31, 120), (32, 120), (54, 280), (63, 300)])
def test_walked_cells_equal_small_calls(K, R):
    from paper_2105_12070_amd import chem
    assert torch.cuda.is_available()
    mech = make_mechanism(K, R, R // 10, R // 20, 7000 + K)
    m = chem.Mechanism(mech)
    st = torch.tensor(make_states(mech, 5003, 41, [(900.0, 2200.0)]), device=DEV)
    f = chem.rhs(m, st, 101325.0)
    J, fj = chem.jacobian(m, st, 101325.0)
    assert torch.isfinite(f).all() and torch.isfinite(J).all()
    for lo in range(0, st.shape[1], 257):
        part = st[:, lo:lo + 257].contiguous()
        assert torch.equal(chem.rhs(m, part, 101325.0), f[:, lo:lo + 257])
        Jp, fp = chem.jacobian(m, part, 101325.0)
        assert torch.equal(Jp, J[lo:lo + 257]) and torch.equal(fp, fj[:, lo:lo + 257])
