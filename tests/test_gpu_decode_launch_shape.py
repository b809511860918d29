"""The decode launch's two shapes: one block per wavefront up to 256 blocks per CU, up to three beyond."""
import pytest

from paper_2604_02715_amd import inputs
from test_gpu_materialize import run_against_model

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [7, 8])
def test_either_side_of_the_line(n):
    # about 8700 blocks an expert (1.411 bytes an element in blocks of 4096): 7 are 61000, 8 are 70000, the line is at 65536 on 256 CUs;
    # sizes that leave a short last block
    cfg = inputs.scaled(inputs.CONFIGS["c1_tiny"], n_experts=8, hidden=4104, ffn=2056, n_slots=8)
    run_against_model(cfg, [(0, [3, 0, 6, 1, 5, 2, 4, 7][:n], [7, 2, 0, 5, 1, 6, 3, 4][:n])])
