"""The compositing forward with a larger scene's ray tiles cut into 4 or 16 parts, and its backward's
items of few tiles: views whose last parts lie past the edge, views narrower than a tile, beside an
uncut scene -- alone, in one batch and without an allocation, against the FP64 oracle (the checks and
tolerances of the two forms' test)."""
from __future__ import annotations

import pytest

from tests import test_gpu_composite_forms as forms
from tests.test_gpu_composite_forms import fmb  # noqa: F401  (the module's fixture)

pytestmark = pytest.mark.gpu

# (Gaussians, views, scale range); 475 tiles in 4 parts, few tiles in 16
CUTS = {
    "four": [(200, [(149, 203)], (0.02, 0.1)), (20, [(16, 16)], (0.05, 0.2))],
    "sixteen": [(600, [(37, 29)], (0.01, 0.05)), (140, [(9, 5), (3, 70)], (0.05, 0.2)), (129, [(8, 8)], (0.05, 0.2))],
}


@pytest.mark.parametrize("label", list(CUTS))
def test_parts(fmb, monkeypatch, label):  # noqa: F811
    monkeypatch.setitem(forms.SETS, label, CUTS[label])
    forms.test_forms_alone_and_mixed(fmb, label)
