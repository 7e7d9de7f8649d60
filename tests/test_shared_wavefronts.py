"""Weight systems solved one to a wavefront and several to a wavefront. Orders
1 to 6 with 8192 or more systems (or nodes) take the second form, all others the
first; both do the same operations on each system, in the same order."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

GROUP_MIN = 8192  # fewest systems that share wavefronts


def moments(m):
    return (m * m + 3 * m) // 2


@pytest.fixture(scope="module")
def dev():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2102_02019_amd import labfm

    labfm.lib()
    return torch.device("cuda:0")


def T(a, dev):
    return torch.from_numpy(np.ascontiguousarray(a)).to(dev)


def bits(t):
    return t.contiguous().view(torch.uint8)


@pytest.mark.parametrize("m", range(1, 11))
def test_solver_holds_the_kernels_of_the_build(m):
    """solve_systems is there to check the pivots of the kernels that build the
    weights: the library has a solve form of each."""
    from paper_2102_02019_amd import labfm

    with open(labfm.LIB_PATH, "rb") as f:
        code = f.read()
    for build, solve, last in (("build_rows_kernel", "rows_solve_kernel", 10),
                               ("build_group_kernel", "group_solve_kernel", 6)):
        if m <= last:
            assert f"{build}ILi{m}E".encode() in code
            assert f"{solve}ILi{m}E".encode() in code


def tie_systems(m):
    """Near ties, exact ties and separated pairs of pivot candidates, with the
    pivot rows that the rule names."""
    from test_gpu_pivot import block_system

    rng = np.random.default_rng(300 + m)
    made = [block_system(moments(m), rng) for _ in range(23)]
    return np.stack([s for s, _, _ in made]), np.stack([p for _, p, _ in made])


# the fewest systems that share wavefronts, with every remainder of four (the
# systems of one wavefront)
@pytest.mark.gpu
@pytest.mark.parametrize("m", [1, 2, 3, 4, 5, 6])
@pytest.mark.parametrize("count", [GROUP_MIN, GROUP_MIN + 1, GROUP_MIN + 2, GROUP_MIN + 3])
def test_pivots_of_systems_sharing_wavefronts(dev, m, count):
    """The pivots are those of the rule, and every solution has the bits that
    the same system's has when it is one of few; a zero column and an infinite
    one among the others mark their own systems alone."""
    from paper_2102_02019_amd import labfm

    few, piv = tie_systems(m)
    n, k = few.shape[1], len(few)
    bad = few[:2].copy()
    bad[0, :, n // 2] = 0.0
    bad[1, :, n // 2] = np.inf
    few, piv = np.concatenate([few, bad]), np.concatenate([piv, np.full((2, n), -1)])
    at = np.random.default_rng(count).integers(0, k + 2, count)
    at[-1], at[-2] = 0, k  # the last system is a good one, beside a singular one
    one = labfm.solve_systems(m, T(few, dev))
    many = labfm.solve_systems(m, T(few, dev)[T(at, dev)])
    status = np.where(np.arange(k + 2) < k, labfm.NODE_OK, labfm.NODE_SINGULAR)
    assert one[2].cpu().numpy().tolist() == status.tolist()
    assert np.array_equal(one[1].cpu().numpy(), piv)
    for a, b in zip(many, one):
        assert torch.equal(bits(a), bits(b[T(at, dev)]))


def node_set(side, dev, **kw):
    from paper_2102_02019_amd import inputs

    nodes = inputs.jittered_lattice(side, seed=side, m=4, **kw)
    return (nodes,) + tuple(T(getattr(nodes, k), dev) for k in ("x", "y", "h", "s"))


H_OVER_S = {1: 1.2, 2: 1.3, 3: 1.4, 4: 1.55, 5: 1.9, 6: 2.2}


@pytest.mark.gpu
@pytest.mark.parametrize("m", [1, 2, 3, 4, 5, 6])
def test_build_does_not_depend_on_the_number_of_nodes(dev, m):
    """A node's weights, float32 copies, kappa, row sums and moments have the
    same bits whether its wavefront is shared or not: all nodes of a set at one
    order, and a third of them, the others at no supported order."""
    from paper_2102_02019_amd import labfm

    nodes, x, y, h, s = node_set(93, dev, h_over_s=H_OVER_S[m])
    assert nodes.n >= GROUP_MIN
    rp, col = labfm.build_neighbours(x, y, h, nodes.box)
    third = np.random.default_rng(m).random(nodes.n) < 1 / 3
    assert 0 < third.sum() < GROUP_MIN
    out = []
    for orders in (np.full(nodes.n, m), np.where(third, m, 0)):
        out.append(labfm.build_weights(x, y, h, s, T(orders.astype(np.int8), dev), nodes.box, rp,
                                       col, f32=True, rowsum=True, tiles=False))
    node = T(third, dev)
    edge = torch.repeat_interleave(node, (rp[1:] - rp[:-1]).long())
    a, b = out
    for pick, names in ((edge, ("w", "w32")), (node, ("rowsum", "mom32", "kappa", "status"))):
        for name in names:
            u, v = getattr(a, name), getattr(b, name)
            assert torch.equal(bits(u[..., pick]), bits(v[..., pick])), name


@pytest.mark.gpu
@pytest.mark.parametrize("m", [1, 4, 5, 6])
@pytest.mark.parametrize("n", [8192, 8195])
def test_each_operator_of_shared_wavefronts(dev, m, n):
    """Each operator's weights and row sums, on their own, against the
    workgroup-per-node build, whose pivots and operation order differ: 1e-9 of
    the weights, above cond(M~) eps at these orders; a row sum is off by no more
    than its weights are together."""
    from paper_2102_02019_amd import labfm

    nodes, x, y, h, s = node_set(93, dev, h_over_s=H_OVER_S[m])
    orders = np.full(nodes.n, 2, np.int8)
    orders[np.random.default_rng(n).permutation(nodes.n)[:n]] = m
    rp, col = labfm.build_neighbours(x, y, h, nodes.box)
    out = []
    for mode in (labfm.BUILD_ROWS, labfm.BUILD_BLOCK):
        labfm.set_build_config(mode)
        try:
            out.append(labfm.build_weights(x, y, h, s, T(orders, dev), nodes.box, rp, col,
                                           rowsum=True, tiles=False))
        finally:
            labfm.set_build_config(0)
    a, b = out
    row = torch.repeat_interleave(torch.arange(nodes.n, device=dev), (rp[1:] - rp[:-1]).long())
    of_m = T(orders == m, dev)
    for k in range(labfm.NUM_OPS):
        scale = torch.zeros(nodes.n, dtype=torch.float64, device=dev)
        scale.index_add_(0, row, b.w[k].abs())
        for nodes_of in (of_m, ~of_m):
            e = nodes_of[row]
            assert torch.linalg.norm((a.w[k] - b.w[k])[e]) <= 1e-9 * torch.linalg.norm(b.w[k][e])
            off = torch.linalg.norm((a.rowsum[k] - b.rowsum[k])[nodes_of])
            assert off <= 1e-9 * torch.linalg.norm(scale[nodes_of])


@pytest.mark.gpu
@pytest.mark.parametrize("m", [1, 2, 3, 4, 5, 6])
def test_optimised_scales_do_not_depend_on_the_number_of_nodes(dev, m):
    """The passes of 16,384 nodes start in the three-operator build of shared
    wavefronts (order 6: two nodes to one, all others four); a third of the
    nodes at a time, the others at order 0, takes the one-node build
    throughout. Each node's scale and count are the same."""
    from paper_2102_02019_amd import labfm

    nodes, x, y, _, s = node_set(128, dev)
    h0 = 2.8 * s
    h, it = labfm.optimise_stencils(x, y, s, m, nodes.box, h0=h0)
    assert int(it.max()) > 10 and int((it > 5).sum()) >= GROUP_MIN
    part = np.random.default_rng(m).integers(0, 3, nodes.n)
    for k in range(3):
        orders = np.where(part == k, m, 0).astype(np.int8)
        assert 0 < (orders == m).sum() < GROUP_MIN
        h1, it1 = labfm.optimise_stencils(x, y, s, T(orders, dev), nodes.box, h0=h0)
        pick = T(part == k, dev)
        assert torch.equal(it1[pick], it[pick]) and torch.equal(h1[pick], h[pick])
