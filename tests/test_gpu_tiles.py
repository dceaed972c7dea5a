"""Kernel edges against the oracle: tile remainders, the smallest and the largest of a
kernel's range, and either side of a dispatch rule."""

import numpy as np
import pytest
import torch

from oracle import exfold_oracle as O
from paper_2608_24938_amd import exfold as X
from paper_2608_24938_amd import synth

from .gpu_common import LayerPair, sync, to_dev

pytestmark = pytest.mark.gpu


def _shape(d, inter, n, k, dtype="f32", shared=0, bias=False):
    return synth.LayerShape("edge", d=d, inter=inter, n_experts=n, top_k=k, dtype=dtype, shared_inter=shared,
                            router_bias=bias)


# Gram tiles of 16 rows: 16, 8, 5 (padded to 8), 3 (padded to 4) and 1 rows a token with ragged token
# counts; more than 16 rows a token (common mode: two tiles a side, the second ragged; nine tiles a side);
# a router bias that gives some experts no token and some several m-tiles of rows.
@pytest.mark.parametrize("n,k,m,mode", [(4, 1, 1, "corouted"), (20, 1, 33, "corouted"), (20, 3, 37, "corouted"),
                                        (24, 5, 131, "corouted"), (64, 8, 301, "corouted"),
                                        (40, 16, 50, "corouted"), (20, 2, 19, "common"), (17, 2, 70, "common"),
                                        (130, 2, 9, "common"), (256, 16, 40, "corouted")])
def test_calibration_at_tile_edges(n, k, m, mode):
    shape = _shape(256, 64, n, k, bias=True)
    lp = LayerPair(shape, seed=n + k)
    xs = synth.calibration_tokens(shape, m, seed=n + k)
    print(f"calibration edge: N={n} K={k} m={m} {mode}", flush=True)
    S, L, h, st = X.calibrate_projectors(lp.dev, to_dev(xs), mode=mode, with_stats=True)
    S2, L2, h2 = X.calibrate_projectors(lp.dev, to_dev(xs), mode=mode)
    sync()
    assert torch.equal(S, S2) and torch.equal(L, L2) and torch.equal(h, h2)
    rS, rL, rh, rst = O.calibrate(lp.ref, synth.widen(xs), k, lam=1e-3, clip=4.0, mode=mode)
    st = st.cpu().numpy()
    np.testing.assert_array_equal(st[..., 3], rst["n"])
    # the expert rows are float32 sums (about 1e-6 each); statistics and scalars are float64 from there
    tol = 1e-4
    for q, key in enumerate("AVC"):
        np.testing.assert_allclose(st[..., q], rst[key], rtol=tol, atol=tol * np.abs(rst[key]).max())
    np.testing.assert_allclose(S.cpu().numpy(), rS, rtol=tol, atol=tol * max(1.0, np.abs(rS).max()))
    obs = rst["n"] > 0
    np.testing.assert_array_equal(L.cpu().numpy()[~obs], rL[~obs])
    np.testing.assert_allclose(L.cpu().numpy()[obs], rL[obs], rtol=tol, atol=tol)
    np.testing.assert_allclose(h.cpu().numpy(), rh, rtol=tol)
