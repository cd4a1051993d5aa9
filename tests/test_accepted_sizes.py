"""Which extents the workspace calls take: every 2,3-smooth one in [2, 512] along
x and y of a 3-D grid, along the last axis (y in 2-D) up to the LDS of its pass.
Tests of the passes pick their lengths from these."""
import pytest

from paper_2003_07720_amd import binding as B

SIZES = [n for n in range(1, 520)]
SMOOTH = [2 ** a * 3 ** b for a in range(10) for b in range(6) if 2 <= 2 ** a * 3 ** b <= 512]
GRIDS = {"x": lambda n: (4, 4, n), "y": lambda n: (4, n, 4), "z": lambda n: (n, 4, 4), "y2d": lambda n: (1, n, 4)}
LAST = {"classical": 256, "polarization": 128}


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("kind", ["classical", "polarization"])
@pytest.mark.parametrize("axis", list(GRIDS))
def test_accepted_extents(axis, kind, prec):
    opts = B.make_options(precision=prec, map=kind)
    for n in SIZES:
        if axis == "z" and n == 1:  # a 2-D grid
            continue
        try:
            B.workspace_size(GRIDS[axis](n), opts)
            taken = True
        except B.RpmError as e:
            assert e.code == -2
            taken = False
        limit = 512 if axis in ("x", "y") else LAST[kind]
        assert taken == (n in SMOOTH and n <= limit), (axis, kind, prec, n)
