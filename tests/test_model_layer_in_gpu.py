"""The layer-in product's column and row blocks (csrc/model.hip): one model step
against the float64 model oracle at each block shape the launch chooses, with
the last row block partly filled, rows wider than one register chunk, rotations
that need wider blocks and an fc1 width that ends inside a block.  Bars as in
test_model_gpu.py."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from test_model_gpu import _gpu, _run_case  # noqa: E402,F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("h,D,d_ff,B,rd", [
    (4, 64, 1024, 17, 16),    # 16 columns x 16 rows, second row block of one row
    (17, 64, 96, 3, 16),      # ... rows wider than a chunk
    (4, 64, 1024, 47, 16),    # 32 columns by grid size
    (4, 64, 96, 5, 32),       # 32 columns for the rotation; fc1 ends inside a head's width
    (4, 64, 1024, 81, 16),    # 64 columns by grid size
    (4, 64, 96, 5, 64),       # 64 columns for the rotation; fc1 ends inside a block
    (4, 64, 1024, 193, 64),   # 64 columns x 32 rows, last row block of one row
    (13, 64, 2080, 100, 64),  # ... rows wider than a chunk
    (16, 64, 4800, 35, 16),   # 64 columns x 16 rows: a third row block of three rows
    (4, 128, 160, 17, 16),    # head dim 128: eight blocks a head
    (4, 128, 96, 17, 128),    # 128 columns; fc1 ends inside a block
    (4, 128, 800, 193, 16),   # 128 columns by grid size; one row in the last block
])
def test_layer_in_blocks_match_oracle(h, D, d_ff, B, rd):
    ctx = np.array([(i * 13) % 70 for i in range(B)], np.int32)
    g = 1 if h <= 16 else h  # at most 16 query heads share a KV head
    _run_case(2, h, D, d_ff, 1, g, B, ctx, seed=500 + h + B + rd, rd=rd,
              label=f"layer-in h{h} D{D} ff{d_ff} B{B} rd{rd}")
