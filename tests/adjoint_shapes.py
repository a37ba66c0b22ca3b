"""Geometries at the edges of the staged adjoint: (volume, detector, projections, offsets).

129, 130 and 131 projections pass the 64-pair table of window origins, with 65 pairs (the
last one half empty, then full) and 66 (half empty): a lone last pair, and a full last
double pair, of the contraction that takes two.  All three are split over blocks.
Detectors smaller than a window, of one row, larger than the volume's shadow; bricks cut
on every axis; voxel pairs (even nx without offsets) and none."""
import numpy as np

import oracle
import tt_inputs as synth
from geoms import tilted_angles

SHAPES = {
    "paired_129": ((8, 9, 10), (11, 12), 129, False),
    "paired_130": ((8, 6, 9), (12, 11), 130, False),
    "paired_131": ((6, 9, 8), (11, 12), 131, False),
    "unpaired_129": ((9, 8, 9), (12, 11), 129, False),
    "offsets_131": ((8, 9, 10), (11, 12), 131, True),
    "detector_below_window": ((10, 6, 9), (5, 4), 9, False),
    "one_detector_row": ((7, 9, 8), (1, 30), 9, True),
    "two_planes": ((2, 17, 3), (6, 21), 15, False),
    "one_projection": ((6, 5, 4), (40, 37), 1, False),
}


def geometry(name, ell, n_seg, model):
    n, (nj, nk), n_proj, offsets = SHAPES[name]
    inner, outer = tilted_angles((n_proj + 2) // 3, (0.0, 27.0, 45.0), span_deg=360.0)
    inner, outer = inner[:n_proj], outer[:n_proj]
    kw = {}
    if offsets:
        kw = dict(joff=np.linspace(-2.0, 3.0, n_proj), koff=np.linspace(1.5, -2.5, n_proj))
    return oracle.Geometry(n, ell, inner, outer, nj, nk, n_seg, synth.lab_frame(), model=model, **kw)
