"""Workspace sizes on grids of odd edge (no GPU): problems at the limit of the static scratch fit it."""
import pytest

M = pytest.importorskip('paper_2412_16638_amd')
A = M._abi


def _bytes(shape, storage, krylov, fmt, tab='SDIRK3', **over):
    op = (A.OP_HEAT, 1.0, (0.0, 0.0, 0.0), A.BC_DIRICHLET0) if krylov == 'cg' \
        else (A.OP_ADVDIFF, 1e-2, (1.0, 0.5, 0.25), A.BC_PERIODIC)
    h = A.mprk_create(A.mprk_grid(*shape, op[3]), A.mprk_operator(op[0], fmt, op[1], (A.C.c_double * 3)(*op[2])),
                      M.tableau(tab), M.precisions(storage, krylov, **over), 1e-3, 0)
    n = A.mprk_workspace_bytes(h)
    A.mprk_destroy(h)
    return n


# (bytes with one value per group: 67103232 and 67105024)
@pytest.mark.parametrize("shape,storage,fmt,over", [((37, 31, 73), 'fp64', A.FMT_CSR, {'restart': 32}),
                                                    ((61, 31, 104), 'fp32', A.FMT_STENCIL, {})])
def test_problems_at_the_scratch_limit_fit(shape, storage, fmt, over):
    assert _bytes(shape, storage, 'gmres', fmt, **over) <= A.STATIC_SCRATCH_BYTES
