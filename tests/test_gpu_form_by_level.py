"""2-D FP32 levels on either side of the sizes where the Dirichlet smoothers go
from the direct form to operator passes: against the FP64 step on the same
values, and the same bits from every workgroup shape."""
import sys

import pytest

from paper_2405_18982_amd import dgmg, inputs

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)


@pytest.mark.parametrize("k,L", [(4, 5), (4, 6), (5, 6), (5, 7), (6, 5), (6, 6)])
@pytest.mark.parametrize("variant", [dgmg.SMOOTH_EXACT, dgmg.SMOOTH_LOCAL])
def test_fp32_step(tmp_path, k, L, variant):
    print(f"form by level k={k} L={L} variant={variant}", flush=True)
    sys.stdout.flush()
    nrhs, E = 3, 2 * (k + 1)
    outs, ref = {}, None
    for shape in (0, 3, 4, 8, 11):
        prob = dgmg.Problem(2, k, L, precision=32, variant=variant, nrhs_max=nrhs)
        cache = tmp_path / f"tune{shape}.json"
        cache.write_text("{\n" + ",\n".join(
            f'  "gfx950/d2/k{k}/L{L}/nrhs{nrhs}/fp32/smooth/l{l}": {{"shape": {shape}, "remap": 1, "us": 1.000}}'
            for l in range(1, L + 1)) + "\n}\n")
        prob.autotune(nrhs=nrhs, cache=str(cache))
        x = torch.from_numpy(inputs.uniform(131, (nrhs, prob.ndofs()))).to("cuda", torch.float32)
        b = torch.from_numpy(inputs.uniform(132, (nrhs, prob.ndofs()))).to("cuda", torch.float32)
        if ref is None:
            ref = [prob.smooth(x.double(), b.double(), reverse=r) for r in (False, True)]
        outs[shape] = [prob.smooth(x.clone(), b, reverse=r) for r in (False, True)] + [prob.vcycle(b)]
        prob.close()
    for got, want in zip(outs[0], ref):
        # rounded coefficients through a patch solve: the root of its condition (about
        # E^4) times the round-off
        err = float((got.double() - want).norm() / want.norm())
        assert err <= E ** 2 * 2.0 ** -24, err
    for shape in (3, 4, 8, 11):
        for got, want in zip(outs[shape], outs[0]):
            assert torch.equal(got, want), shape
