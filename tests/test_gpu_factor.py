"""The supernodal factor and L_ss^-1 against the FP64 oracle on boxes whose supernodes sit at the edges of the 16-column
blocks, 64-column tiles, 256-column panels and doubling steps: from a single partial tile to several panels, flat, long
and two-component meshes.

W_H = H A^-1 H^T of every surface node runs through all of the factor; the bar is the 1e-10 of the other parity tests."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle.icr_oracle as O  # noqa: E402
from paper_2306_06946_amd.scenes import box_grid  # noqa: E402

pytestmark = pytest.mark.gpu


def _scene(grids, seed):
    rng = np.random.default_rng(seed)
    nodes, tets, fixed, surf, shift = [], [], [], [], 0.0
    for nx, ny, nz in grids:
        x, t, ijk = box_grid(nx, ny, nz, 0.01, 0.2, rng)
        base = sum(len(a) for a in nodes)
        nodes.append(x + np.array([shift, 0.0, 0.0]))
        shift += 0.01 * (nx + 3)
        tets.append(t + base)
        fixed.append(ijk[:, 2] == nz - 1)
        surf.append(np.any((ijk == 0) | (ijk == np.array([nx, ny, nz]) - 1), axis=1))
    tets = np.concatenate(tets).astype(np.int32)
    fixed, surf = np.concatenate(fixed), np.concatenate(surf)
    return dict(nodes=np.concatenate(nodes), tets=tets, E=np.exp(rng.uniform(np.log(1e3), np.log(1e5), len(tets))),
                nu_e=np.full(len(tets), 0.45), rho=1e3, alpha=0.1, beta=0.1, h=0.01, gravity=np.array([0, 0, -9.81]),
                fixed=fixed.astype(np.uint8), free_surface=np.nonzero(surf & ~fixed)[0])


@pytest.mark.parametrize("grids", [
    [(2, 2, 2)], [(3, 2, 2)], [(4, 4, 3)], [(5, 4, 3)],          # one supernode: 24, 36, 144, 180 columns at most
    [(7, 7, 4)], [(9, 8, 7)], [(6, 5, 31)], [(17, 16, 3)],       # two to four tiles at the root
    [(12, 11, 10)], [(16, 10, 12)], [(17, 17, 8)],               # more than one panel
    [(5, 5, 5), (8, 7, 6)], [(2, 2, 2), (2, 2, 2)],              # two components
], ids=str)
def test_factor_at_tile_and_panel_edges(grids):
    from paper_2306_06946_amd import icr
    sc = _scene(grids, 5)
    pick = sc["free_surface"][:: max(1, len(sc["free_surface"]) // 150)].astype(np.int32)
    asm = O.assemble(sc)
    ref = O.build_WH(O.CholeskyFactor(asm["A"]), pick, asm["n"])
    print(f"[gpu] factor {grids}: {asm['n']} DOF, {len(pick)} contacts", flush=True)
    s = icr.Scene()
    s.assemble(sc)
    s.factor()
    WH = torch.empty(9 * len(pick) ** 2, dtype=torch.float64, device="cuda")
    s.build_WH(torch.from_numpy(pick).cuda(), WH)
    got = WH.cpu().numpy().reshape(ref.shape)
    assert np.linalg.norm(got - ref) <= 1e-10 * np.linalg.norm(ref)
    s.factor()   # again, into the same scene
    s.build_WH(torch.from_numpy(pick).cuda(), WH)
    assert np.array_equal(WH.cpu().numpy().reshape(ref.shape), got)
