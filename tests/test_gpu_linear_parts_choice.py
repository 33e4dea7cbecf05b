"""Plain linear layers of a long K where the choice between the wave-level kernel, the tiles and parts of K turns: seven and eight rows of
fragments (eight parts), nine (whole), thirteen and sixteen (five), seventeen (four), nineteen and more (whole)."""
import pytest

from test_gpu_linear_parts_few import test_linear_packed_parts_few_tokens as run

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M", [193, 256, 257, 385, 512, 513, 577, 704, 768])
def test_linear_packed_parts_of_middle_sizes(M):
    run(M, 1280, 5120)
