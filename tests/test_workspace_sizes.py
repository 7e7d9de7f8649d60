"""Workspaces that users' memory has to hold beside operators of the same size
(no GPU needed)."""
import pytest

from paper_2102_02019_amd import labfm


@pytest.mark.parametrize("n", [1, 1001, 4_194_304])
@pytest.mark.parametrize("steps,every", [(0, 1), (1, 20), (10, 5), (200, 20)])
def test_adjoint_registers_share_their_memory(n, steps, every):
    """Beside the checkpoints and one recomputed segment (three doubles per node
    each) a reversed step holds 60 doubles per node: values that are not live
    together lie in the same place."""
    states = -(-steps // every) + every
    need = labfm.lib().labfm_adjoint_workspace_bytes(n, steps, every)
    assert 8 * n * (3 * states + 60) <= need <= 8 * n * (3 * states + 60) + 512
