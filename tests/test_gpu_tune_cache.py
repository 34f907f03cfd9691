"""One tuning cache for several smoothers: an entry holds for the smoother it was
timed with and for the kernels it was timed on; entries that name neither hold
for every smoother that has none of its own."""
import json

import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2405_18982_amd import dgmg  # noqa: E402

L = 2


def tune(cache, variant):
    print(f"tune cache variant={variant}", flush=True)
    prob = dgmg.Problem(3, 3, L, variant=variant)
    rep = prob.autotune(cache=str(cache)).strip().splitlines()
    prob.close()
    assert len(rep) == 1 + L
    return rep[0], rep[1:]  # the apply, the smoother by level


def test_variants_do_not_share_smoother_entries(tmp_path):
    cache = tmp_path / "tune.json"
    apply_c, smooth_c = tune(cache, dgmg.SMOOTH_CLAMPED)
    assert "(cached)" not in apply_c + "".join(smooth_c)
    apply_e, smooth_e = tune(cache, dgmg.SMOOTH_EXACT)
    assert "(cached)" in apply_e  # one operator for all
    assert not any("(cached)" in ln for ln in smooth_e)
    for variant, first in ((dgmg.SMOOTH_CLAMPED, smooth_c), (dgmg.SMOOTH_EXACT, smooth_e)):
        again = tune(cache, variant)[1]
        assert [ln.replace(" (cached)", "") for ln in again] == first and all("(cached)" in ln for ln in again)
    text = cache.read_text()
    assert text.count('"shape"') == 1 + 2 * L  # both kept, each once


def test_entries_of_other_kernels_are_timed_again(tmp_path):
    cache = tmp_path / "tune.json"
    tune(cache, dgmg.SMOOTH_EXACT)
    rev = [ln for ln in cache.read_text().splitlines() if '"rev"' in ln]
    assert len(rev) == 1 + L
    cache.write_text(cache.read_text().replace('"rev": ', '"rev": 9'))
    apply_l, smooth_l = tune(cache, dgmg.SMOOTH_EXACT)
    assert "(cached)" not in apply_l + "".join(smooth_l)
    assert cache.read_text().count('"shape"') == 1 + L  # in place of the outdated ones
    assert len(json.loads(cache.read_text())) == 1 + L


def test_plain_entries_hold_for_every_variant(tmp_path):
    cache = tmp_path / "tune.json"
    keys = ["apply"] + [f"smooth/l{l}" for l in range(1, L + 1)]
    cache.write_text("{\n" + ",\n".join(
        f'  "gfx950/d3/k3/L{L}/nrhs1/fp64/{key}": {{"shape": 1, "remap": 0, "us": 1.000}}' for key in keys) + "\n}\n")
    for variant in (dgmg.SMOOTH_EXACT, dgmg.SMOOTH_FULL):
        apply_l, smooth_l = tune(cache, variant)
        assert all("shape=1 remap=0" in ln and "(cached)" in ln for ln in [apply_l] + smooth_l)
