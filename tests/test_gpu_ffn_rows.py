"""GPU parity of the walking 256 x 256 tiles that are taken row by row (experts of about one row tile, few column tiles), against the FP64
oracle: more tiles than workgroups, so that workgroups walk on, column tiles that do not divide an XCD's 32, and a few tiles only."""
import pytest

from paper_2604_02715_amd import inputs
from test_gpu_ffn import run_ffn_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kw", [
    dict(n_experts=64, n_slots=64, tokens=8000, top_k=2, hidden=512, ffn=576, routing="uniform"),      # 5 and 2 column tiles, 250 rows each
    dict(n_experts=60, n_slots=60, tokens=6000, top_k=3, hidden=320, ffn=704, routing="zipf"),         # row tiles of 1 to 256 rows, up to dozens for an expert
    dict(n_experts=3, n_slots=3, tokens=520, top_k=1, hidden=128, ffn=64, routing="uniform"),          # one column tile each, fewer tiles than XCDs
])
def test_tiles_row_by_row(kw):
    run_ffn_case(inputs.scaled(inputs.CONFIGS["c1_tiny"], **kw), seed=31)
