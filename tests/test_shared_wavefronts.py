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
