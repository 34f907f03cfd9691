"""The Dirichlet smoothers in direct form (one solve for a patch's new values
from the load, its dropped end nodes and the outer traces) against the oracle's
residual form, and the FP32 operator on differences.

Meshes of 4 cells a direction (every patch touches the boundary; the patch
types of one launch differ within a wave where patches share one) and of 8
(interior patches take their own path), every degree on either side of the
rule that chooses the form, both residuals and orders, a right-hand-side count
that no workgroup shape divides."""
import sys

import numpy as np
import pytest

from oracle.smoother import FDSmoother
from paper_2405_18982_amd import inputs

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2405_18982_amd import dgmg  # noqa: E402


def note(msg):
    print(msg, flush=True)
    sys.stdout.flush()


CASES = [(2, k, L) for k in (3, 4, 5, 6, 7) for L in (1, 2)] + [(3, 1, 2), (3, 2, 2), (3, 3, 2)] + \
        [(3, k, 1) for k in (2, 3, 4, 5, 6, 7)]


@pytest.mark.parametrize("dim,k,L", CASES)
@pytest.mark.parametrize("variant", [dgmg.SMOOTH_EXACT, dgmg.SMOOTH_LOCAL])
def test_direct_form_is_the_residual_form(dim, k, L, variant):
    note(f"direct smoother d={dim} k={k} L={L} variant={variant}")
    N, nrhs, E = 2 ** (L + 1), 3, 2 * (k + 1)
    fs = FDSmoother(dim, k, N, inputs.sigma_of(k), mode="exact" if variant == dgmg.SMOOTH_EXACT else "local")
    n = (N * (k + 1)) ** dim
    X, B = inputs.uniform(91, (nrhs, n)), inputs.uniform(92, (nrhs, n))
    # a value passes 2 dim contractions of E terms per colour (unit round-off
    # u) and the patch eigenpairs, known to u times the condition of the 1-D
    # patch matrix (about E^4 / 2)
    for dt, u in ((torch.float64, 1.1e-16), (torch.float32, 6e-8)):
        tol = 2 * dim * E * u if dt == torch.float32 else max(1e-12, E ** 4 * u)
        prob = dgmg.Problem(dim, k, L, variant=variant, nrhs_max=nrhs)
        Xt, Bt = (torch.from_numpy(v).to("cuda", dt) for v in (X, B))
        X64, B64 = Xt.double().cpu().numpy(), Bt.double().cpu().numpy()
        for reverse in (False, True):
            got = prob.smooth(Xt.clone(), Bt, reverse=reverse).double().cpu().numpy()
            order = list(range(2 ** dim))[::-1 if reverse else 1]
            for j in range(nrhs):
                ref = fs.step(X64[j], B64[j], order)
                assert np.linalg.norm(got[j] - ref) <= tol * np.linalg.norm(ref), (dt, reverse, j)
        prob.close()


@pytest.mark.parametrize("dim,k", [(2, 1), (2, 4), (2, 7), (3, 1), (3, 3), (3, 4), (3, 6), (3, 7)])
def test_fp32_operator_on_constants(dim, k):
    """A times a constant vanishes on cells that no domain face touches.  On
    differences FP32 leaves only the rounding of the tangential masses in the
    jumps: (n + 2) round-offs of a row sum (at most the largest weight, below
    1/2), times the penalty, times the masses of the other directions, on 2 dim
    faces."""
    note(f"fp32 constants d={dim} k={k}")
    L, n = 2, k + 1
    N = 2 ** (L + 1)
    prob = dgmg.Problem(dim, k, L)
    x = torch.full((prob.ndofs(),), 0.7, dtype=torch.float32, device="cuda")
    y = prob.apply(x).cpu().numpy().reshape((N,) * dim + (-1,))
    inner = y[(slice(1, N - 1),) * dim]
    bound = 2 * dim * (n + 2) * 6e-8 * inputs.sigma_of(k) * 0.5 ** (dim - 1) * 0.7 * (1.0 / N) ** (dim - 2)
    assert np.abs(inner).max() <= bound
    prob.close()
