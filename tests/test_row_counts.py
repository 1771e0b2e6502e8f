"""Row counts of the network's entry points up to the largest an int32 holds."""
import pytest

import paper_2407_06042_amd as dm

FULL_GRID = 256 * 4992 * 4   # bytes: one partial gradient of every workgroup


@pytest.mark.parametrize("n", [16384, 65536, 2 ** 31 - 17, 2 ** 31 - 16, 2 ** 31 - 15, 2 ** 31 - 2, 2 ** 31 - 1])
def test_training_workspace_up_to_the_last_row_count(n):
    assert dm.lib().dmala_mlp_train_workspace_size(n) == FULL_GRID


def test_training_workspace_grows_with_the_rows():
    size = dm.lib().dmala_mlp_train_workspace_size
    sizes = [size(n) for n in (1, 64, 65, 1000, 16320, 16321, 16384, 16385)]
    assert sizes == sorted(sizes) and sizes[0] >= 4992 * 4 and sizes[-1] == FULL_GRID
