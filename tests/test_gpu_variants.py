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


# one more and one less than the nodes of a wavefront, several wavefronts; 6 is
# the last order with several systems per wavefront
@pytest.mark.parametrize("m", [1, 2, 3, 4, 5, 6, 7])
@pytest.mark.parametrize("count", [1, 3, 4, 5, 9])
def test_systems_sharing_a_wavefront(dev, m, count):
    """Systems solved side by side in a wavefront do not touch each other: the
    last wavefront's missing systems, and a singular or non-finite system
    among others. Diagonally dominant systems: numpy's solution to 1e-13 (n
    eps times a condition number below 10)."""
    from paper_2102_02019_amd import labfm

    n = (m * m + 3 * m) // 2
    rng = np.random.default_rng(10 * m + count)
    S = rng.uniform(-1.0, 1.0, (count, n, n + 6))
    S[:, :, :n] += 2.0 * n * np.eye(n)[rng.permutation(n)]
    bad = {1: 0.0, 3: np.inf} if count > 3 else {}
    for k, v in bad.items():
        S[k, :, n // 2] = v
    psi, piv, st = (t.cpu().numpy() for t in labfm.solve_systems(m, T(S, dev)))
    for k in range(count):
        if k in bad:
            assert st[k] == labfm.NODE_SINGULAR
            assert (psi[k] == 0.0).all() and (piv[k] == -1).all()
            continue
        assert st[k] == labfm.NODE_OK
        assert sorted(piv[k]) == list(range(n))
        ref = np.linalg.solve(S[k, :, :n], S[k, :, n:])
        assert np.abs(psi[k] - ref).max() <= 1e-13 * np.abs(ref).max()


@pytest.mark.parametrize("m", [1, 4, 5, 6])
@pytest.mark.parametrize("n", [8191, 8192, 8193, 8195])
def test_shared_wavefront_build_matches_workgroup_build(dev, m, n):
    """Around the fewest nodes of an order that share wavefronts (8192), all
    remainders of four but two: weights, kappa, row sums and statuses of the
    default build against the workgroup-per-node build, whose pivots and
    operation order differ: 1e-9 relative, above cond(M~) eps at these
    orders."""
    from paper_2102_02019_amd import labfm

    nodes = inputs.jittered_lattice(93, seed=m, m=4, h_over_s={1: 1.2, 4: 1.55, 5: 1.9, 6: 2.2}[m])
    nodes.m = np.full(nodes.n, 2, np.int8)
    nodes.m[np.random.default_rng(n).permutation(nodes.n)[:n]] = m
    x, y, h, s, mm = (T(getattr(nodes, k), dev) for k in ("x", "y", "h", "s", "m"))
    rp, col = labfm.build_neighbours(x, y, h, nodes.box)
    out = []
    for mode in (labfm.BUILD_ROWS, labfm.BUILD_BLOCK):
        labfm.set_build_config(mode)
        try:
            out.append(labfm.build_weights(x, y, h, s, mm, nodes.box, rp, col, rowsum=True))
        finally:
            labfm.set_build_config(0)
    a, b = out
    assert torch.equal(a.status, b.status)
    for u, v in ((a.w, b.w), (a.kappa, b.kappa), (a.rowsum, b.rowsum)):
        assert torch.linalg.norm(u - v) <= 1e-9 * torch.linalg.norm(v)


def brute_rows(x, y, h, box):
    """Row lengths and columns of the stencils from all pairs, in torch: every
    product and sum rounded on its own, as the predicate demands."""
    n = x.numel()
    cols, lens = [], []

    def wrap(d, L, on):
        if not on:
            return d
        return torch.where(d > 0.5 * L, d - L, torch.where(d < -0.5 * L, d + L, d))

    for i in torch.arange(n, device=x.device).split(max(1, 40_000_000 // n)):
        dx = wrap(x[None, :] - x[i, None], box.Lx, box.periodic_x)
        dy = wrap(y[None, :] - y[i, None], box.Ly, box.periodic_y)
        r = 2.0 * h[i]
        near = dx * dx + dy * dy <= (r * r)[:, None]
        near[torch.arange(i.numel()), i] = False
        lens.append(near.sum(1))
        cols.append(near.nonzero()[:, 1])
    return torch.cat(lens), torch.cat(cols)


# sets around the sizes at which a workgroup's share changes and its last one
# is partly filled; grids of one, two, three and five cells an axis; blocks of
# more candidates than fit in LDS (768), within one cell and over several
@pytest.mark.parametrize("n,cells,spread,px,py", [
    (1, 4, 1.0, True, True), (15, 1, 1.0, False, False), (17, 2, 1.0, True, False),
    (600, 3, 1.0, True, True), (700, 1, 1.0, False, False), (3000, 5, 1.0, False, True),
    (5000, 12, 0.05, True, True), (5000, 12, 0.25, True, True), (4001, 2, 1.0, True, True),
    (16383, 40, 1.0, True, True), (16385, 40, 1.0, False, False), (65535, 90, 1.0, True, True),
    (65599, 90, 0.6, True, False)])
def test_stencil_search_against_all_pairs(dev, n, cells, spread, px, py):
    """Rows bit-exact and ascending; `spread` gathers the nodes into that
    share of the box, across its corner."""
    from paper_2102_02019_amd import labfm

    rng = np.random.default_rng(n + cells)
    box = inputs.Box(2.0, 1.5, px, py)
    x = np.mod(rng.uniform(-0.5, 0.5, n) * spread * box.Lx + (0 if px else 1.0), box.Lx)
    y = np.mod(rng.uniform(-0.5, 0.5, n) * spread * box.Ly + (0 if py else 0.75), box.Ly)
    hmax = 0.2499 * min(box.Lx, box.Ly) if cells <= 2 else box.Ly / (2.01 * cells)
    x, y, h = (T(a, dev) for a in (x, y, hmax * rng.uniform(0.3, 1.0, n)))
    rp, col = labfm.build_neighbours(x, y, h, box)
    lens, ref = brute_rows(x, y, h, box)
    assert torch.equal(rp[1:].long() - rp[:-1].long(), lens) and int(rp[0]) == 0
    assert torch.equal(col.long(), ref)


@pytest.mark.parametrize("side,orders", [(9, (6,)), (17, (1, 2, 4, 11)), (16, (3, 6, 10))])
def test_optimised_scales_do_not_depend_on_company(dev, side, orders):
    """A node's optimised scale is its own: sets whose passes are cut down to
    few nodes of several orders give each node what it gets when the others
    are left out (order 0, which keeps h0)."""
    from paper_2102_02019_amd import labfm

    nodes = inputs.jittered_lattice(side, seed=side, m=4)
    rng = np.random.default_rng(side)
    m = rng.choice(np.array(orders, np.int8), nodes.n)
    x, y, s = T(nodes.x, dev), T(nodes.y, dev), T(nodes.s, dev)
    h0 = 1.9 * s
    h, it = labfm.optimise_stencils(x, y, s, T(m, dev), nodes.box, h0=h0)
    assert (it >= 0).all() and torch.equal(h[it == 0], h0[it == 0])
    assert (it[T(m, dev) == 11] == 0).all()
    some = rng.random(nodes.n) < 0.3
    h1, it1 = labfm.optimise_stencils(x, y, s, T(np.where(some, m, 0).astype(np.int8), dev),
                                      nodes.box, h0=h0)
    some = T(some, dev)
    assert torch.equal(h1[some], h[some]) and torch.equal(it1[some], it[some])
    assert (it1[~some] == 0).all()


# an odd and an even number of stencil entries, and transposed weights that
# start 8 bytes off a pair: the three ways the transposed gathers load edges;
# steps that fill the last segment, leave it short, or make one segment
@pytest.mark.parametrize("odd", [False, True])
@pytest.mark.parametrize("steps,ckpt,filt", [(1, 3, True), (4, 2, True), (5, 2, False), (3, 7, True)])
def test_adjoint_against_differences(dev, odd, steps, ckpt, filt):
    """<J v, w> from central differences of the run (step 1e-6: truncation
    about 1e-11, rounding 1e-9 of the product) against <v, J^T w>; the
    misaligned weights give the aligned ones' result to rounding."""
    from paper_2102_02019_amd import labfm

    prm = inputs.taylor_green_params()
    for seed in range(1, 100):
        nodes = inputs.jittered_lattice(17, seed=seed, m=4)
        nodes.h = nodes.h * np.random.default_rng(seed).uniform(0.95, 1.05, nodes.n)
        x, y, h, s = (T(getattr(nodes, k), dev) for k in ("x", "y", "h", "s"))
        rp, col = labfm.build_neighbours(x, y, h, nodes.box)
        if col.numel() % 2 == int(odd):
            break
    ops = labfm.build_weights(x, y, h, s, 4, nodes.box, rp, col, rowsum=True)
    assert ops.nnz % 2 == int(odd)
    rng = np.random.default_rng(5)
    rho, u, v = inputs.taylor_green_state(nodes.x, nodes.y)
    q0 = T(np.concatenate([np.log(rho), u, v]), dev)
    vec, bar = T(rng.standard_normal(3 * nodes.n), dev), T(rng.standard_normal(3 * nodes.n), dev)
    dt, eps = 0.05 * float(nodes.s[0]), 1e-6
    ends = []
    for sign in (1.0, -1.0):
        q = q0 + sign * eps * vec
        labfm.rk_step(q, ops, prm, dt, steps, filter=filt)
        ends.append(q)
    jv = float(torch.dot((ends[0] - ends[1]) / (2.0 * eps), bar))
    grad = labfm.rk_adjoint(q0, bar, ops, prm, dt, steps, ckpt_every=ckpt, filter=filt)
    scale = float(torch.linalg.norm(grad) * torch.linalg.norm(vec))
    assert abs(jv - float(torch.dot(vec, grad))) <= 1e-7 * scale
    tptr, tsrc, tw = ops.transpose
    off = torch.empty(tw.numel() + 1, dtype=tw.dtype, device=dev)[1:]
    off.copy_(tw)
    ops.transpose = (tptr, tsrc, off)
    again = labfm.rk_adjoint(q0, bar, ops, prm, dt, steps, ckpt_every=ckpt, filter=filt)
    assert torch.linalg.norm(again - grad) <= 1e-13 * torch.linalg.norm(grad)
    ops.transpose, ops.use_tiles = (tptr, tsrc, tw), False
    again = labfm.rk_adjoint(q0, bar, ops, prm, dt, steps, ckpt_every=ckpt, filter=filt)
    assert torch.linalg.norm(again - grad) <= 1e-12 * torch.linalg.norm(grad)


# 16 lanes take 32 edges a pass, 32 lanes 64, or 96 where the mean exceeds 64,
# 8 lanes 32, 4 lanes 16: rows around each; none, one and several operators
@pytest.mark.parametrize("rows", [(0, 1, 3, 15, 16, 17, 4), (0, 31, 32, 33, 63, 64, 65, 2),
                                  (95, 96, 97, 191, 0, 193, 1)])
@pytest.mark.parametrize("prec_name", ["F64", "F32W", "F32_COMP"])
def test_operator_subsets_and_row_lengths(dev, rows, prec_name):
    """Every number of operators and every lane count against numpy, within the
    rounding of a sum of K products: 2 K eps of the summed magnitudes, (K eps32)^2
    times four for the compensated float32 sums."""
    from paper_2102_02019_amd import labfm

    prec = getattr(labfm, prec_name)
    rng = np.random.default_rng(17)
    cnt = np.array(rows * 3 + rows[:2])
    n, rp = cnt.size, np.concatenate([[0], np.cumsum(cnt)])
    nnz, kmax = int(rp[-1]), int(cnt.max())
    col = rng.integers(0, n, nnz)
    w, phi = rng.standard_normal((6, nnz)), rng.standard_normal(n)
    mom = (1e-3 * rng.standard_normal((6, n))).astype(np.float32)
    stride = int(labfm.lib().labfm_w32_stride(nnz))
    w32 = torch.zeros((6, stride), dtype=torch.float32, device=dev)
    w32[:, :nnz] = T(w.astype(np.float32), dev)
    ops = labfm.Operators(T(rp.astype(np.int32), dev), T(col.astype(np.int32), dev), T(w, dev),
                          w32[:, :nnz], T(np.zeros(n), dev), mom32=T(mom, dev))
    f32 = prec_name != "F64"
    wd = (w.astype(np.float32) if f32 else w).astype(np.float64)
    d = phi[col] - np.repeat(phi, cnt)
    row = np.repeat(np.arange(n), cnt)
    ref, mag = np.zeros((6, n)), np.zeros((6, n))
    for k in range(6):
        np.add.at(ref[k], row, wd[k] * d)
        np.add.at(mag[k], row, np.abs(wd[k] * d))
    if f32:
        for k in (2, 3, 4):
            mx, my = mom[2 * (k - 2)].astype(np.float64), mom[2 * (k - 2) + 1].astype(np.float64)
            ref[k] -= ref[0] * mx + ref[1] * my
            mag[k] += mag[0] * np.abs(mx) + mag[1] * np.abs(my)
    eps = 2 * (kmax + 4) * 2.0 ** -53
    if prec_name == "F32_COMP":
        eps += 4 * ((kmax + 4) * 2.0 ** -24) ** 2
    try:
        for lpn in (0, 4, 8, 16, 32):
            labfm.set_launch_config(labfm.KERNEL_APPLY, prec, lpn, 0)
            for mask in (0x01, 0x20, 0x10, 0x06, 0x1C, 0x2D, 0x1F, 0x3F):
                got = labfm.apply_operators(ops, T(phi, dev), mask, prec).cpu().numpy()
                sel = [k for k in range(6) if mask >> k & 1]
                bad = np.abs(got.reshape(len(sel), n) - ref[sel]) > eps * mag[sel]
                assert not bad.any(), (lpn, hex(mask))
    finally:
        labfm.set_launch_config(labfm.KERNEL_APPLY, prec, 0, 0)


# distinct neighbours of the first tile: one, around a group of four, around
# the workgroup's 256 threads, the capacity, and one and many past it; the
# second tile holds one node
@pytest.mark.parametrize("distinct", [1, 4, 5, 255, 257, 1023, 1024, 1025, 3000])
@pytest.mark.parametrize("step", [1, 2048])
def test_tile_halos(dev, distinct, step):
    """The halo is the sorted set of a tile's neighbours and every entry finds
    its own index through it; consecutive and widely spaced indices (runs in
    the hash table), each neighbour listed up to four times."""
    from paper_2102_02019_amd import labfm

    n = labfm.TILE_NODES + 1
    rng = np.random.default_rng(distinct + step)
    base = step * np.arange(distinct, dtype=np.int64) + 7
    first = rng.permutation(np.concatenate([base, base[::2], base[::2], base[:3]]))
    cuts = np.sort(rng.integers(0, first.size + 1, labfm.TILE_NODES - 1))
    rp = np.concatenate([[0], cuts, [first.size, first.size + 2]])
    col = np.concatenate([first, [5, 3]])
    ops = labfm.Operators(T(rp.astype(np.int32), dev), T(col.astype(np.int32), dev), None, None,
                          torch.zeros(n, dtype=torch.float64, device=dev))
    ok = labfm.build_tiles(ops)
    assert ok == (distinct <= labfm.TILE_HALO_MAX)
    if not ok:
        return
    hc, hi, lc, hmax = (v.cpu().numpy() if torch.is_tensor(v) else v for v in ops.tiles)
    halo = hi.reshape(2, -1)
    assert hc.tolist() == [distinct, 2] and hmax == max(distinct, 2)
    assert np.array_equal(halo[0, :distinct], base) and halo[1, :2].tolist() == [3, 5]
    assert np.array_equal(halo[0, lc[:first.size]], first) and lc[first.size:].tolist() == [1, 0]


# the neighbours in reach shrink from pass to pass (the lists start at some 130
# and 190 entries: several rounds of 64, the last ones partly filled)
@pytest.mark.parametrize("m,side", [(4, 23), (6, 33)])
@pytest.mark.parametrize("wide", [1.2, 1.5])
def test_optimisation_drops_neighbours_out_of_reach(dev, m, side, wide):
    """Entries beyond 2 h carry zero weights, so a CSR that lists more of them
    gives every node the same scale and count."""
    import ctypes

    from paper_2102_02019_amd import labfm

    nodes = inputs.jittered_lattice(side, seed=side, m=m)
    x, y, s = T(nodes.x, dev), T(nodes.y, dev), T(nodes.s, dev)
    mt = torch.full((nodes.n,), m, dtype=torch.int8, device=dev)
    h0 = (2.2 if m == 4 else 2.8) * s
    h, it = labfm.optimise_stencils(x, y, s, m, nodes.box, h0=h0)
    rp, col = labfm.build_neighbours(x, y, wide * h0, nodes.box)
    h1, it1 = torch.empty_like(h), torch.empty_like(it)
    ws = torch.empty(labfm.lib().labfm_optimise_workspace_bytes(nodes.n, col.numel()),
                     dtype=torch.uint8, device=dev)
    prm = labfm._StencilOptParams(0.99, 1.01, 1e4, 200)
    code = labfm.lib().labfm_optimise_stencils(
        x.data_ptr(), y.data_ptr(), h0.data_ptr(), s.data_ptr(), mt.data_ptr(), nodes.n,
        labfm._box(nodes.box), rp.data_ptr(), col.data_ptr(), col.numel(), ctypes.byref(prm),
        h1.data_ptr(), it1.data_ptr(), ws.data_ptr(), ws.numel(),
        torch.cuda.current_stream().cuda_stream)
    assert code == labfm.OK
    assert int(it.max()) > 10
    assert torch.equal(it, it1) and torch.equal(h, h1)
