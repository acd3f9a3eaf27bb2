"""The Courant numbers where a wave takes several short rows and where a long
row is cut among waves: rows of 4 to 32 cells (a power of two and one off it)
whose count does not fill the last wave, rows one cell past a piece, many pieces
of few rows, and the most rows that are cut and one more.
The bar is that of test_gpu_courant.py."""
import pytest

import test_gpu_courant as whole
from paper_2004_13887_amd import inputs as I

pytestmark = pytest.mark.gpu

SIZES = [(3, 5, 4, False), (3, 7, 5, False), (5, 5, 8, True), (3, 3, 9, False), (4, 7, 16, True), (3, 7, 17, False),
         (3, 3, 31, False), (5, 3, 32, True), (20, 400, 7, True), (3, 3, 33, False), (3, 3, 257, False),
         (4, 5, 513, True), (3, 3, 60000, False), (32, 32, 257, False), (25, 41, 257, False)]


@pytest.mark.parametrize("nr,nt,np_,sphere", SIZES)
@pytest.mark.parametrize("where", [0, -1])
def test_maxima_in_any_piece(nr, nt, np_, sphere, where):
    spec = I.full_sphere(nr, nt, np_) if sphere else I.sector(nr, nt, np_, 1e-4, 1e-5)
    whole.test_maxima_anywhere(spec, where)
