"""The batch draw on either side of the line between its forms (500 (draws - 4) atoms, at
least 8,192 and at most 32,768), against the oracle's batches rank for rank."""
import pytest

pytestmark = pytest.mark.gpu

pytest.importorskip("torch")


@pytest.mark.parametrize("n,p_shell,box", [(8191, 12, 8.0), (8192, 12, 8.0), (32767, 70, 12.0), (32768, 70, 12.0)])
def test_draws_on_either_side(orc, n, p_shell, box):
    from test_gpu_draw_forms import _compare
    _compare(orc, n, box, 0.8, 1.2, p_shell, [3, 1 << 34])
