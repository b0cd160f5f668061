"""Sizes at the edges of kernel tiles and of the rules that choose between kernels, against
the float64 oracle under the gates of tests/gpu_util.py."""
import pytest

from bpt_inputs import make_inputs, small_workload
from gpu_util import run_gpu, run_oracle, say
from test_gpu_parity import compare_all

pytestmark = pytest.mark.gpu


# fp32: attention blocks of 16 rows shared by 4 waves (S around 16 and 64, one token), GEMM
# tiles of 32, 64 and 128 (the largest from 256 tiles of 128 x 128 on: the FFN of the last case)
@pytest.mark.parametrize("B,S,D,H,F,causal", [
    (1, 1, 128, 2, 64, True), (3, 15, 128, 1, 192, True), (2, 17, 192, 3, 256, False), (1, 65, 256, 2, 320, True),
    (2, 129, 128, 2, 512, False), (1, 1100, 512, 4, 1024, True), (1, 2048, 256, 2, 2048, True)])
def test_f32_tile_edges(B, S, D, H, F, causal):
    w = small_workload("f32", B=B, S=S, D=D, H=H, F=F, causal=causal, Bq=min(S, 64), Bkv=min(S, 64))
    inp = make_inputs(w, seed=3, affine=True, biases=True)
    say(f"case {w.name}")
    gpu = run_gpu(w, inp, qkv_grads=True)
    Yr, _, g = run_oracle(w, inp)
    compare_all(w, inp, gpu, Yr, g, "fp32", w.name)
