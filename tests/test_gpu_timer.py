"""The launch timer's names as the header lists them, and the attention path that the widths take."""

import os
import re

import numpy as np
import pytest
import torch

from paper_2608_16305_amd import mtgnn as M
from paper_2608_16305_amd.step import TGNStep
from synth import init_params, make_stream, workload
from tests._gpu import log, needs_gpu
from tests.test_gpu_attn import _forward_backward

pytestmark = [pytest.mark.gpu, needs_gpu]

QUERY_NAMES = ("attn_fwd", "attn_bwd", "attn_dw")
SLOT_NAMES = ("gemm_kv_proj", "k_attn_core", "k_attn_core_bwd", "gemm_kv_dw", "gemm_kv_dx")
MERGE_NAMES = ("merge_fwd", "merge_bwd", "dw_os")
STEP_NAMES = ("gru_fused", "gemm_gru_dw", "link_fused", "dw_os")


def _launches(name, call):
    M.timer_start(name, 64)
    try:
        call()
    finally:
        ms, n = M.timer_stop()
    assert n == 0 or ms > 0
    return n


def _attention(H, width, de, k, dtype):
    bf16 = dtype == "bf16"
    store = torch.bfloat16 if bf16 else torch.float32
    gen = torch.Generator().manual_seed(3)
    u = lambda *s: torch.rand(*s, generator=gen) * 2 - 1   # noqa: E731
    w, kv, Q = width, 2 * width + de, 40
    p = {n: (u(*s) * 0.1).to(store) for n, s in dict(W_q=(w, 2 * w), W_k=(w, kv), W_v=(w, kv), W_o=(w, w), W_1=(w, 2 * w),
                                                     W_2=(w, w)).items()}
    p.update({"b" + n[1:]: u(w) for n in list(p)})
    ids = lambda hi, *s: torch.randint(0, hi, s, generator=gen, dtype=torch.int32)   # noqa: E731
    args = (p, u(50, w).to(store), u(60, de) if de else None, ids(50, Q), u(Q), ids(50, Q, k), u(Q, k), ids(60, Q, k), u(w),
            u(w), u(Q, w), H, k, torch.arange(50, dtype=torch.int32), bf16)
    return lambda: _forward_backward(*args)


def test_header_lists_the_names():
    text = open(os.path.join(os.path.dirname(__file__), "..", "include", "mtgnn.h")).read()
    part = text[text.index("/* Launch timer"):text.index("mtgnn_timer_stop waits")]
    assert set(re.findall(r'"(\w+)"', part)) == {*QUERY_NAMES, *SLOT_NAMES, *MERGE_NAMES, *STEP_NAMES, "gemm"}


#        H  width edge k   by query
ROUTES = [(2, 100, 16, 5, True), (1, 32, 0, 1, True),
          (2, 128, 0, 1, True), (2, 128, 1, 1, False), (2, 128, 1, 2, True),       # rows to and past 128
          (1, 128, 128, 1, True), (1, 128, 129, 1, False), (1, 128, 129, 2, True),   # to and past 256, one head
          (2, 128, 128, 2, True), (2, 100, 157, 3, False), (2, 100, 157, 4, True),   # two heads: k d_attn >= 400
          (2, 32, 256, 12, False), (2, 32, 256, 13, True),
          (4, 100, 16, 5, False), (2, 30, 0, 5, False), (1, 64, 257, 20, False)]


@pytest.mark.parametrize("H,width,de,k,by_query", ROUTES)
def test_attention_route(H, width, de, k, by_query):
    log(f"[timer] heads {H}, width {width}, edge {de}, k {k}")
    call = _attention(H, width, de, k, "f32")
    got = {n: _launches(n, call) for n in QUERY_NAMES + SLOT_NAMES}
    log("  " + ", ".join(f"{n} {v}" for n, v in got.items()))
    assert all((got[n] > 0) == by_query for n in QUERY_NAMES), got
    assert all((got[n] > 0) != by_query for n in SLOT_NAMES), got


def test_other_names_have_launches():
    call = _attention(4, 100, 0, 5, "f32")
    got = {n: _launches(n, call) for n in MERGE_NAMES}
    got["gemm"] = _launches("gemm", _attention(4, 100, 0, 5, "bf16"))
    w = workload(1)
    s = make_stream(w)
    r = TGNStep(w, s, init_params(w, random_bias=True), np.zeros((w.n_nodes, w.d_mem), np.float32),
                np.zeros(w.n_nodes, np.float32))
    r.step(1)
    for n in STEP_NAMES:
        got[n] = got.get(n, 0) + _launches(n, lambda: r.step(2))
    torch.cuda.synchronize()
    log("[timer] " + ", ".join(f"{n} {v}" for n, v in got.items()))
    assert all(v > 0 for v in got.values()), got
