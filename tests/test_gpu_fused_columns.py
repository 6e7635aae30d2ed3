"""The fused kernel's column layouts and chunk edges, through the C ABI.

Groups of up to eight heads share one MFMA between the hi and mid terms of a
query and split the row's tiles between the halves of the columns; larger
groups use a column per head.  Sessions go to their units in chunks of 64
tokens.  Every layout is compared with the multi-kernel path, which does
neither, at sizes around a tile, a chunk and a unit.
"""
import numpy as np
import pytest
import torch

from paper_2607_10582_amd import binding as B

from harness import REL
from test_gpu_tail_groups import run

pytestmark = pytest.mark.gpu

# one token joins each session at each of the two steps
EDGES = [1, 14, 15, 16, 62, 63, 64, 65, 127, 254, 255, 256, 257, 511, 600, 1025]


@pytest.fixture(autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a ROCm device")
    B.load_library()


@pytest.mark.parametrize("L,Hq,Hkv,P,kw", [
    (1, 1, 1, 16, {}),                  # one row, one column
    (3, 3, 1, 64, {}),
    (3, 8, 2, 16, {}),                  # four heads
    (4, 10, 2, 64, {}),                 # five heads, both halves in use
    (9, 12, 2, 16, {}),                 # more rows than the ring holds
    (2, 8, 1, 16, {}),                  # eight heads: the last packed layout
    (2, 9, 1, 16, {}),                  # nine: a column per head
    (2, 16, 1, 64, {}),
    (3, 8, 2, 16, {"window": 2}),       # packed columns of two queries
    (3, 12, 2, 16, {"window": 2}),      # a column per head and query
    (3, 12, 2, 16, {"aligned": True}),
    (3, 12, 2, 64, {"quant": 10.0}),
    (3, 12, 1, 16, {"quant": 10.0}),
    (3, 8, 2, 16, {"window": 2, "aligned": True, "quant": 10.0}),
])
def test_fused_agrees_with_the_multi_kernel_path(L, Hq, Hkv, P, kw):
    a, ca = run(EDGES, L, Hq, Hkv, P, True, **kw)
    b, cb = run(EDGES, L, Hq, Hkv, P, True, fused=False, **kw)
    assert ca["first_fused"] and not cb["first_fused"]
    for step, (x, y) in enumerate(zip(a, b)):
        for u, v in zip(x[:3], y[:3]):
            assert np.array_equal(np.isfinite(u), np.isfinite(v))
            fin = np.isfinite(v)
            np.testing.assert_allclose(u[fin], v[fin], rtol=REL, atol=1e-30, err_msg=f"step {step}")
        assert np.array_equal(x[3], y[3])
    assert abs(float(a[0][0].sum()) - len(EDGES)) < 1e-3 * len(EDGES)
    print(f"[{L}x{Hq}/{Hkv} P={P} {kw}] ok", flush=True)
