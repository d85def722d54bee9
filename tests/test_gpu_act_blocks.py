"""np_act_batch at the edges of its block choice: each block (128 x 256, 128 x
128, 64 x 128 and 64 x 64 neurons x tokens, the last two with one token block
and with several), ragged neuron and token counts, widths that end inside a
128- or 256-byte piece, every type.  Dyadic records (m 2^-6, |m| <= 3) and
tokens in {-4..4}: every sum is exact in fp32 in any order, so the activations
must equal the exact values (ReLU-gated), whatever the block."""
import numpy as np
import pytest
import torch

import oracle as orc
from paper_2608_22643_amd import binding as B
from paper_2608_22643_amd import workload as W
from gpu_util import DEV, say, to_dev

pytestmark = pytest.mark.gpu

CASES = [  # (type, d, F, n): the block the rule takes
    ("f16", 136, 14300, 500),   # 128 x 256
    ("bf16", 64, 14336, 513),   # 128 x 256, one token in the last block
    ("f16", 200, 14001, 250),   # 128 x 128
    ("bf16", 128, 2000, 1500),  # 128 x 128
    ("f16", 264, 14000, 127),   # 64 x 128, one token block
    ("bf16", 8, 14336, 128),    # 64 x 128, one iteration
    ("bf16", 384, 7001, 200),   # 64 x 128, two token blocks
    ("f16", 520, 1001, 64),     # 64 x 64, one token block
    ("bf16", 256, 65, 1),       # 64 x 64, one token
    ("f16", 72, 3002, 300),     # 64 x 64, several token blocks
    ("f32", 36, 14336, 512),    # 128 x 256
    ("f32", 68, 14333, 256),    # 128 x 128
    ("f32", 100, 9001, 129),    # 64 x 128 or 64 x 64
    ("f32", 4, 50, 17),         # 64 x 64
]


@pytest.mark.parametrize("dt,d,F,n", CASES, ids=[f"{c[0]}_d{c[1]}_F{c[2]}_n{c[3]}" for c in CASES])
def test_act_blocks_exact(dt, d, F, n):
    cfg = W.Config("act_blocks", 1, d, F, 8, 1 / F, 1 / F, dt, dt, n, rho_given=0.0, k_override=1,
                   c_override=1, dyadic=True, dyadic_w_range=3, dyadic_h_range=4)
    say(f"[act blocks] {dt} d {d} F {F} n {n}")
    shape = B.make_shape(1, d, F, 8, 1, 1, dt, dt, "relu")
    store, h = W.storage(cfg)[0], W.hidden(cfg, n)
    acts = torch.full((n, F), float("nan"), dtype=torch.float32, device=DEV)
    B.np_act_batch(shape, to_dev(store), to_dev(h), n, acts)
    torch.cuda.synchronize()
    rec, x = orc.decode(dt, store), orc.decode(dt, h)
    g, u = x @ rec[:, :d].T, x @ rec[:, d:2 * d].T
    ref = np.maximum(g, 0) * u
    assert np.max(np.abs(ref)) < 2.0 ** 12
    assert np.array_equal(acts.cpu().numpy().astype(np.float64), ref)
