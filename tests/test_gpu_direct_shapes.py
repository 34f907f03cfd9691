"""The direct smoothers in every way the tuner can launch them, against the
oracle's residual form: several patches in a wave (2-D shape 0), one patch a
workgroup (2-D shape 4; two waves a patch in 3-D Q3 and Q7), several right-hand
sides of one patch with the last workgroup partly empty (8, 9).  A mesh of 8 cells
has boundary patches and, in every colour, interior ones, which take the passes
of a type known at compile time wherever a wave holds one type only."""
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


@pytest.mark.parametrize("dim,k,L", [(2, 4, 2), (2, 5, 2), (2, 6, 2), (2, 7, 2), (3, 2, 2), (3, 3, 2), (3, 4, 2), (3, 7, 1)])
@pytest.mark.parametrize("variant", [dgmg.SMOOTH_EXACT, dgmg.SMOOTH_LOCAL])
@pytest.mark.parametrize("bits", [64, 32])
def test_shapes_against_the_oracle(tmp_path, dim, k, L, variant, bits):
    print(f"direct shapes d={dim} k={k} variant={variant} fp{bits}", flush=True)
    sys.stdout.flush()
    N, nrhs, E = 2 ** (L + 1), 3, 2 * (k + 1)
    dt, u = (torch.float64, 2.0 ** -53) if bits == 64 else (torch.float32, 2.0 ** -24)
    fs = FDSmoother(dim, k, N, inputs.sigma_of(k), mode="exact" if variant == dgmg.SMOOTH_EXACT else "local")
    n = (N * (k + 1)) ** dim
    X, B = (torch.from_numpy(inputs.uniform(s, (nrhs, n))).to("cuda", dt) for s in (141, 142))
    x64, b64 = X.double().cpu().numpy(), B.double().cpu().numpy()
    # 2 dim contractions of E terms a colour; in FP64 the oracle's own 1-D data,
    # known to the condition of the patch matrix, about E^4 / 2
    tol = 2 * dim * E * u if bits == 32 else max(1e-12, E ** 4 * u)
    for reverse in (False, True):
        order = list(range(2 ** dim))[::-1 if reverse else 1]
        ref = [fs.step(x64[j], b64[j], order) for j in range(nrhs)]
        first = None
        for shape in (0, 4, 5, 8, 9):
            prob = dgmg.Problem(dim, k, L, precision=bits, variant=variant, nrhs_max=nrhs)
            cache = tmp_path / f"tune{shape}.json"
            cache.write_text("{\n" + ",\n".join(
                f'  "gfx950/d{dim}/k{k}/L{L}/nrhs{nrhs}/fp{bits}/smooth/l{l}": '
                f'{{"shape": {shape}, "remap": 0, "us": 1.000}}' for l in range(1, L + 1)) + "\n}\n")
            prob.autotune(nrhs=nrhs, cache=str(cache))
            got = prob.smooth(X.clone(), B, reverse=reverse)
            out = got.double().cpu().numpy()
            for j in range(nrhs):
                assert np.linalg.norm(out[j] - ref[j]) <= tol * np.linalg.norm(ref[j]), (shape, reverse, j)
            first = got if first is None else first
            assert torch.equal(got, first), (shape, reverse)
            prob.close()
