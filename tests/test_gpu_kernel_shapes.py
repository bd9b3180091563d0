"""GPU parity at the sizes where the kernels' tiles, cuts and dispatch rules change over, against the float64 oracle with
the bounds of test_gpu_parity."""
import pytest

from paper_2510_03515_amd import workloads as wl
from test_gpu_parity import _check_pair, _run_pair, rb  # noqa: F401  (rb is the library fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,V,prompts,length", [
    (50, 1000, 11, 65),     # logits in 64 x 64 tiles with remainders, dHidden and dW in 16 x 16 tiles, contraction shared out
    (260, 1100, 11, 65),    # dHidden and dW in 32 x 32 tiles
    (520, 3700, 2, 10),     # dW in 64 x 64 tiles, logits in 32 x 32 tiles, fewer rows than a step of the contraction
    (3, 17, 1, 2),          # everything smaller than one tile and one step
])
@pytest.mark.parametrize("layout", ["dv", "vd"])
@pytest.mark.parametrize("min_ws", [False, True])
def test_fp64_matrix_tiles(rb, d, V, prompts, length, layout, min_ws):
    print(f"fp64 tiles d {d} V {V} rows {prompts * 3 * length} {layout} min_ws {min_ws}", flush=True)
    spec = wl.small_spec("f64_tiles", "f32", d=d, V=V, prompts=prompts, G=3, len_lo=max(1, length - 3), len_hi=length, reward="uniform")
    w, out, ref = _run_pair(rb, spec, layout=layout, min_ws=min_ws)
    _check_pair(rb, spec, out, ref, layout)
