"""W_H against the FP64 oracle at the contact counts where the tile size of the multi-RHS products changes and at the
edges of both tile sizes, overlapped or on one stream.  The bar is the 1e-10 of the other parity tests."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle.icr_oracle as O  # noqa: E402
from paper_2306_06946_amd.scenes import box_grid  # noqa: E402

pytestmark = pytest.mark.gpu

_CACHE = {}


def _box(grid):
    if grid not in _CACHE:
        rng = np.random.default_rng(3)
        x, t, ijk = box_grid(*grid, 0.01, 0.2, rng)
        fixed = ijk[:, 2] == grid[2] - 1
        surf = np.any((ijk == 0) | (ijk == np.array(grid) - 1), axis=1)
        sc = dict(nodes=x, tets=t.astype(np.int32), E=np.full(len(t), 1e4), nu_e=np.full(len(t), 0.45), rho=1e3,
                  alpha=0.1, beta=0.1, h=0.01, gravity=np.array([0, 0, -9.81]), fixed=fixed.astype(np.uint8))
        asm = O.assemble(sc)
        _CACHE[grid] = sc, rng.permutation(np.nonzero(surf & ~fixed)[0]).astype(np.int32), O.CholeskyFactor(asm["A"]), asm["n"]
    return _CACHE[grid]


@pytest.mark.parametrize("overlap", [True, False])
@pytest.mark.parametrize("grid,counts", [
    ((9, 8, 7), (1, 10, 11, 21, 22, 43, 85)),           # last column tile of 1 to 64 columns
    ((20, 19, 8), (341, 427, 661, 662, 824)),   # Z^T Z of the root on both sides of 512 tiles of 64 (31 and 32 a side)
], ids=str)
def test_wh_at_tile_edges(grid, counts, overlap):
    from paper_2306_06946_amd import icr
    sc, surf, fac, n = _box(grid)
    s = icr.Scene()
    s.assemble(sc)
    s.factor()
    s.set_overlap(overlap)
    for c in counts:
        pick = np.ascontiguousarray(surf[:c])
        assert len(pick) == c
        print(f"[gpu] W_H tiles {grid} {c} overlap {overlap}", flush=True)
        ref = O.build_WH(fac, pick, n)
        WH = torch.empty(9 * c * c, dtype=torch.float64, device="cuda")
        s.build_WH(torch.from_numpy(pick).cuda(), WH)
        got = WH.cpu().numpy().reshape(ref.shape)
        assert np.linalg.norm(got - ref) <= 1e-10 * np.linalg.norm(ref)
        assert np.array_equal(got, got.T)
