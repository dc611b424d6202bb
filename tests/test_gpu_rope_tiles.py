"""RoPE and the cache append in the tiled GEMM's epilogue: prompts whose QKV projection takes each kind of tile (one to
eight row blocks of a wavefront; row positions loaded before the products and behind them), with last row blocks
that are not full and sequences that start inside one; the generation step behind it reads what was appended."""
import pytest

import synth
from test_gpu_tiled_gemm import run

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rows", [18, 41, 100, 143, 190, 250, 300, 450, 590, 639, 720, 900, 1100, 1180])
def test_prompt_and_step(rows):
    shape = synth.StageShape("bf16", 1, 256, 16, 16, 128, 256, 0)
    first = rows // 2 + 1
    run(shape, [first, rows - first - 5, 5], 1, rows)


@pytest.mark.parametrize("rows", [60, 333])
def test_heads_of_64_columns_grouped(rows):
    run(synth.StageShape("bf16", 1, 256, 12, 3, 64, 256, 0), [rows - 9, 9], 1, rows)
