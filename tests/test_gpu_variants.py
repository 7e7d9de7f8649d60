"""Kernel variants at the sizes where they can go wrong: remainders of tiles
and workgroups, the smallest sets, odd counts. References are the general
kernels of the library or plain numpy."""
import numpy as np
import pytest

from paper_2102_02019_amd import inputs

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dev():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2102_02019_amd import labfm

    labfm.lib()
    return torch.device("cuda:0")


def T(a, dev):
    return torch.from_numpy(np.ascontiguousarray(a)).to(dev)


def lattice(side, m, dev, seed=3, **kw):
    """Operators, node tensors and a smooth state of a jittered lattice."""
    from paper_2102_02019_amd import labfm

    nodes = inputs.jittered_lattice(side, seed=seed, m=m)
    x, y, h, s = (T(getattr(nodes, k), dev) for k in ("x", "y", "h", "s"))
    rp, col = labfm.build_neighbours(x, y, h, nodes.box)
    ops = labfm.build_weights(x, y, h, s, m, nodes.box, rp, col, **kw)
    rho, u, v = inputs.taylor_green_state(nodes.x, nodes.y)
    p = inputs.fourier_perturbation(nodes.x, nodes.y, seed=seed)
    q = np.concatenate([np.log(rho) + p[0], u + p[1], v + p[2]])
    return nodes, ops, T(q, dev)


# 81 nodes: two whole tiles of 32 and one of 17; 1089: 34 and one node; 1024:
# whole tiles only
@pytest.mark.parametrize("side", [9, 32, 33])
@pytest.mark.parametrize("prec_name", ["F64", "F32W", "F32_COMP"])
def test_alternating_tile_order(dev, side, prec_name):
    """The tiled launches of a step sweep the tiles upwards and downwards in
    turn: every node is updated once per launch, so three steps agree with the
    untiled kernels to rounding (1e-14 per step's sums of ~30 terms), and graph
    replay equals eager stepping bitwise."""
    from paper_2102_02019_amd import labfm

    prec = getattr(labfm, prec_name)
    prm = inputs.taylor_green_params()
    nodes, ops, q0 = lattice(side, 4, dev, f32=True)
    out = {}
    for name, tiles, graph in (("tiled", True, False), ("graph", True, True),
                               ("untiled", False, False)):
        ops.use_tiles = tiles
        q = q0.clone()
        labfm.rk_step(q, ops, prm, 0.05 * float(nodes.s[0]), 3, prec=prec, use_graph=graph)
        out[name] = q.cpu().numpy()
    assert np.isfinite(out["tiled"]).all()
    assert np.array_equal(out["tiled"], out["graph"])
    d = np.linalg.norm(out["tiled"] - out["untiled"]) / np.linalg.norm(out["untiled"])
    assert d <= 3e-14
