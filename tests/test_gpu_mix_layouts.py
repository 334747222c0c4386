"""Residual mixing at the edges of its launch rules: rows of one chunk up to more columns than a
block has waves, lanes and waves that end part-way, token counts around the XCD windows."""
import numpy as np
import pytest
import torch

import workloads
from tests._gpu import say
from tests.test_gpu_mix import check_case
from tests.test_gpu_n8 import gauss8

pytestmark = pytest.mark.gpu

# chunks of 16 bytes per row, tokens: the short rows (8, 16 and 32 lanes per token), one column
# (four tokens per block), several, and turns of the block's waves or shares of the row
ROWS = [(1, 70), (7, 33), (8, 64), (9, 31), (16, 40), (17, 9), (32, 300), (33, 257), (63, 5), (64, 130), (65, 129),
        (129, 128), (257, 127), (320, 3), (512, 136), (513, 20), (768, 17), (1024, 9), (1025, 5), (2100, 2)]


@pytest.mark.parametrize("n", [4, 8])
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("nc,B", ROWS, ids=[f"{c}x{b}" for c, b in ROWS])
def test_rows(n, dtype, nc, B):
    C = nc * (8 if dtype == torch.bfloat16 else 4)
    say(f"test: mixing layouts, n={n} {dtype} C={C} ({nc} chunks), B={B}")
    rng = np.random.default_rng([n, nc, B])
    H = workloads.gauss(B, 3.0, seed=nc)[0] if n == 4 else gauss8(B, 3.0, nc)[0]
    X = rng.standard_normal((B, n, C), dtype=np.float32)
    G = rng.standard_normal((B, n, C), dtype=np.float32)
    if dtype == torch.bfloat16:
        X, G = (workloads.bf16_to_f32(workloads.bf16_bits(v)) for v in (X, G))
    check_case(H, X, G, dtype, f"n={n} nc={nc} B={B}")
