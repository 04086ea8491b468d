"""Host logic of bench.py's profile summaries, on synthetic rocprofv3 kernel
traces whose kernel durations are known: every (loop, layer, kernel) average
and every span must come out exactly."""
import csv
import os
import sys

import pytest

sys.path.insert(0, os.path.dirname(os.path.dirname(os.path.abspath(__file__))))
import bench  # noqa: E402

R, J = 3, 2  # loops, layers of the synthetic runs


class Trace:
    """Kernels laid end to end with a fixed gap; timestamps in ns."""

    def __init__(self, gap_ns=1000):
        self.rows, self.t, self.gap = [], 0, gap_ns

    def add(self, name, us):
        start = self.t + self.gap
        end = start + int(round(us * 1e3))
        self.rows.append({"Kernel_Name": name, "Start_Timestamp": str(start), "End_Timestamp": str(end)})
        self.t = end

    def write(self, path):
        rows = list(self.rows)
        rows.reverse()  # the summaries sort by start time themselves
        with open(path, "w", newline="") as f:
            w = csv.DictWriter(f, fieldnames=["Kernel_Name", "Start_Timestamp", "End_Timestamp"])
            w.writeheader()
            w.writerows(rows)


# the prefill kernels of bf16 models, and of float32 models and few rows
PRE = {"qkv": "k_pgemm<1, A_SRC, E_QKV, false>", "attn": "k_attn_prefill<bf16, 64, false, 8>",
       "o": "k_pgemm<1, A_CMP, E_RESID, false>", "gate_up": "k_pgemm<1, A_SRC, E_SWIGLU, false>",
       "down": "k_pgemm<1, A_CMP, E_RESID, false>"}
PRE_F32 = {"qkv": "k_gemm<float, E_QKV>", "attn": "k_attn_prefill<float, 64, true, 8>", "o": "k_gemm<float, E_RESID>",
           "gate_up": "k_gemm<float, E_SWIGLU>", "down": "k_gemm<float, E_RESID>"}
PRE_FEW = {"qkv": "k_dgemm<bf16, E_QKV>", "attn": "k_attn_prefill<bf16, 64, true, 4>", "o": "k_dgemm<bf16, E_RESID>",
           "gate_up": "k_dgemm<bf16, E_SWIGLU>", "down": "k_dgemm<bf16, E_RESID>"}
HEADS = {"dgemm": "k_dgemm<bf16, E_LOGITS>", "pgemm": "k_pgemm<2, A_SRC, E_LOGITS, false>", "gemm": "k_gemm<float, E_LOGITS>"}


def pre_us(p, i, j, kind):
    """Duration of kernel `kind` at loop i, layer j of prefill p."""
    return 10.0 * (1 + list(PRE).index(kind)) + 3.0 * i + 0.5 * j + 0.25 * p


def add_prefill(tr, p, names=PRE, head=HEADS["dgemm"]):
    tr.add("k_fill_i32", 1.0)
    tr.add("k_embed_route<bf16>", 5.0)
    tr.add("k_plan_count", 1.5)
    tr.add("k_plan_prefill", 0.5)
    for i in range(R):
        for j in range(J):
            tr.add(names["qkv"], pre_us(p, i, j, "qkv"))
            tr.add(names["attn"], pre_us(p, i, j, "attn"))
            tr.add(names["o"], pre_us(p, i, j, "o"))
            tr.add("k_resid_norm<1>", 1.0)
            tr.add(names["gate_up"], pre_us(p, i, j, "gate_up"))
            tr.add(names["down"], pre_us(p, i, j, "down"))
            tr.add("k_resid_norm<1>", 1.0)
    tr.add(head, 4.0)


FORMS = [(PRE, "dgemm"), (PRE, "pgemm"), (PRE_F32, "dgemm"), (PRE_F32, "gemm"), (PRE_FEW, "dgemm")]
FORM_IDS = ["bf16", "bf16-many-logits", "f32", "f32-many-logits", "few-rows"]


@pytest.mark.parametrize("names,head", FORMS, ids=FORM_IDS)
def test_prefill_trace_summary(tmp_path, names, head):
    tr = Trace()
    for p in range(4):  # a warm-up prefill, then three timed ones
        add_prefill(tr, p, names, HEADS[head])
    for _ in range(3):
        tr.add("__amd_rocclr_copyBuffer", 50.0)  # host copies after the session
    for p in range(4, 6):  # the next session
        add_prefill(tr, p, names, HEADS[head])
    path = tmp_path / "trace.csv"
    tr.write(path)
    out = bench.prefill_trace_summary(str(path), R, J, first=1, count=3)
    assert out["prefills"] == [1, 4]
    for i, row in enumerate(out["per_loop_us"]):
        assert row["loop"] == i + 1
        for kind in PRE:
            want = sum(pre_us(p, i, j, kind) for p in (1, 2, 3) for j in range(J)) / (3 * J)
            assert row[kind] == pytest.approx(want, abs=1e-9), (i, kind)
    for kind in PRE:
        want = sum(pre_us(p, i, j, kind) for p in (1, 2, 3) for i in range(R) for j in range(J)) / 3
        assert out["per_prefill_us"][kind] == pytest.approx(want, abs=1e-9), kind
    # span: the first kernel after the previous prefill's head to this
    # prefill's head, gaps included (one gap per kernel), never the copies
    kernels = 4 + R * J * 7 + 1
    busy = [1.0 + 5.0 + 2.0 + 4.0 + sum(pre_us(p, i, j, k) for i in range(R) for j in range(J) for k in PRE)
            + R * J * 2 * 1.0 for p in (1, 2, 3)]
    want = sum(b + (kernels - 1) * 1.0 for b in busy) / 3
    assert out["span_us"] == pytest.approx(want, abs=1e-6)


@pytest.mark.parametrize("names,head", FORMS, ids=FORM_IDS)
def test_mfma_summary(tmp_path, names, head):
    """Two sessions of four prefills; the set-up kernels between them and the
    copies after the last belong to no prefill."""
    tr = Trace()
    for p in range(8):
        if p == 4:
            tr.add("__amd_rocclr_copyBuffer", 50.0)
            tr.add("k_wfrag<bf16>", 70.0)
        add_prefill(tr, p, names, HEADS[head])
    tr.add("__amd_rocclr_copyBuffer", 50.0)
    path = tmp_path / "counters.csv"
    util = lambda n: 40.0 if "gemm" in n else 20.0 if "attn" in n else 0.0  # noqa: E731
    with open(path, "w", newline="") as f:
        w = csv.DictWriter(f, fieldnames=["Dispatch_Id", "Kernel_Name", "Start_Timestamp", "End_Timestamp",
                                          "Counter_Name", "Counter_Value"])
        w.writeheader()
        for k, r in enumerate(tr.rows):
            us = (int(r["End_Timestamp"]) - int(r["Start_Timestamp"])) / 1e3
            for c, v in (("MfmaUtil", util(r["Kernel_Name"])), ("MfmaFlopsBF16", 1e6 * us)):
                w.writerow(dict(r, Dispatch_Id=k + 1, Counter_Name=c, Counter_Value=v))
    out = bench.mfma_summary(str(path))
    for label, first in (("one_part", 1), ("hi_lo_parts", 5)):
        got, ps = out[label], range(first, first + 3)
        block = {k: sum(pre_us(p, i, j, k) for p in ps for i in range(R) for j in range(J)) / 3 for k in PRE}
        total = sum(block.values()) + 1.0 + 5.0 + 2.0 + 4.0 + R * J * 2 * 1.0
        assert got["ms_per_prefill"] == pytest.approx(total / 1e3, abs=1e-9)
        busy = 40.0 * (total - 8.0 - R * J * 2 * 1.0 - block["attn"]) + 20.0 * block["attn"]
        assert got["mfma_busy_pct"] == pytest.approx(busy / total, abs=1e-9)
        assert got["executed_tflop_per_prefill"] == pytest.approx(total * 1e-6, abs=1e-12)


DEC = ("qkv", "attn", "o", "gate_up", "down")
DEC_NAME = {"qkv": "k_dgemm<E_QKV>", "attn": "k_attn_decode<bf16, 64, 4>", "o": "k_dgemm<E_RESID>",
            "gate_up": "k_dgemm<E_SWIGLU>", "down": "k_dgemm<E_RESID>"}


def dec_us(st, i, j, kind):
    return 5.0 * (1 + DEC.index(kind)) + 2.0 * i + 0.5 * j + 0.125 * st


def test_decode_trace_summary(tmp_path):
    steps = 6
    tr = Trace()
    for st in range(steps):
        tr.add("k_embed_route<bf16>", 3.0)
        tr.add("k_plan_decode", 2.0)
        for i in range(R):
            for j in range(J):
                for kind in DEC:
                    tr.add(DEC_NAME[kind], dec_us(st, i, j, kind))
        tr.add("k_gemm<E_LOGITS>", 7.0)
        tr.add("k_argmax_finalize", 1.0)
    path = tmp_path / "trace.csv"
    tr.write(path)
    per_step = R * J
    out = bench.trace_summary(str(path), routed_launches=steps * per_step, last_dispatches=2 * per_step,
                              loops=R, layers=J, first_step=1, last_step=4)
    # the attention average over the last two steps' launches
    want = sum(dec_us(st, i, j, "attn") for st in (4, 5) for i in range(R) for j in range(J)) / (2 * per_step)
    assert out["attn_routed_timed_region"]["dispatches"] == 2 * per_step
    assert out["attn_routed_timed_region"]["avg_us"] == pytest.approx(want, abs=1e-9)
    table = {(t["loop"], t["layer"]): t for t in out["decode_steps"]["per_loop_layer_us"]}
    for i in range(R):
        for j in range(J):
            for kind in DEC:
                want = sum(dec_us(st, i, j, kind) for st in (1, 2, 3)) / 3
                assert table[(i + 1, j + 1)][kind] == pytest.approx(want, abs=1e-9), (i, j, kind)
    # a step's span runs from its embedding kernel to the kernel before the
    # next step's embedding kernel; every kernel after the first adds one gap
    kernels = 2 + per_step * 5 + 2
    busy = [3.0 + 2.0 + 7.0 + 1.0 + sum(dec_us(st, i, j, k) for i in range(R) for j in range(J) for k in DEC)
            for st in (1, 2, 3)]
    assert out["decode_steps"]["span_us"] == pytest.approx(sum(busy) / 3 + (kernels - 1) * 1.0, abs=1e-6)
    assert out["decode_steps"]["gaps_us"] == pytest.approx((kernels - 1) * 1.0, abs=1e-6)
