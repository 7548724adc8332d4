"""Both sides of the lines between the tail's one launch and its split form: 12 and 13 draft tokens, 16 with 4 and 5 windows, 512 and 513
windows; with the judge's scores compared."""
import pytest

import workloads as wl
from parity import parity_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,K", [(3, 12), (3, 13), (4, 16), (5, 16), (512, 2), (513, 2)])
@pytest.mark.parametrize("dtype,d_t", [("bf16", 256), ("f32", 64)])
def test_tail_forms(B, K, dtype, d_t):
    base = "tiny_f32" if dtype == "f32" else "8b_b1_k16"
    w = wl.scaled(wl.WORKLOADS[base], name="tail", p_match=0.6, B=B, K=K, d_t=d_t, d_d=64, V=600)
    rep, x, draft, greedy, gpu = parity_case(w, 31, repeat=2)
    assert rep["near_thr_windows"] <= 1 + B // 100
