"""The contact search's cell table against the oracle at the sizes where its
level, the blocks' remainders and the search below a table cell change. Labels
and counts are whole numbers: the bar is equality."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

# bodies (8^k and its neighbours: the table takes one level more; 1024 and 4096:
# the wide blocks and the one-block build end), radius in units of the mean spacing
SIZES = (1, 2, 8, 9, 64, 65, 512, 513, 1024, 1025, 4096, 4097)
RADII = (0.0, 1e-4, 0.3, 40.0)


@pytest.mark.parametrize("scale", RADII)
@pytest.mark.parametrize("n", SIZES)
def test_cell_table_edges(n, scale):
    from paper_1912_04197_amd import api

    rng = np.random.default_rng(1000 + n)
    # half uniform, half in a clump a thousand times smaller: cells of the table
    # hold from no body to half of them
    pos = rng.random((n, 3))
    pos[: n // 2] = 0.25 + 1e-3 * pos[: n // 2]
    if n > 64:
        pos[5] = pos[17]
    if scale == 40.0 and n > 1025:
        pytest.skip("every pair touches: quadratic on both sides")
    r = scale * n ** (-1.0 / 3.0) * (0.5 + 0.5 * rng.random(n))
    want_label, want_contacts, want_sets = oracle.contact_components(pos, r, 0.0)
    ctx = api.Context(n)
    dev = [torch.from_numpy(np.ascontiguousarray(a)).cuda() for a in (pos, np.ones(n) / n, r)]
    for _ in range(2):  # the table is left over from the first pass in the second
        label, contacts, sets = ctx.contact_components(*dev, 0.0)
        assert (contacts, sets) == (want_contacts, want_sets)
        assert np.array_equal(label.cpu().numpy(), want_label)
