"""The colouring asks for the memory it always asked for: a caller that keeps the
size of one call for the next library is not refused."""
import pytest

from paper_2212_00574_amd.binding import kz_colour_workspace_bytes


@pytest.mark.parametrize("n,most", [(1, 1280), (64, 1280), (65, 1792), (511, 5120), (512, 5120), (1000, 9728),
                                    (3000, 44288), (20000, 552192), (65536, 1877248)])
def test_no_more_than_before(n, most):
    assert kz_colour_workspace_bytes(n) <= most
