#!/usr/bin/env python3
"""Throughput of the FL-GLM server stack on one MI355X.

One step = the server's whole hot path over one client batch: forward through
the N server blocks, then backward (returning every client's input gradient
and accumulating fp32 weight gradients), all through the C ABI
(fl_server_stack_forward / fl_server_stack_backward).  Inputs are resident in
HBM before the timed region; weights, activations and upstream gradients are
seeded synthetic draws with the workload's shapes and distributions.

Prints one JSON line: tokens/s of the whole step, the fraction of the bf16
matrix-core peak it reaches, a per-kernel-class breakdown (HIP events around
every launch of one untimed step after the warmup), the roofline entry of the
dominant kernel class (its launches timed with events during the timed
steps, the only ones that carry events there), and the CPU oracle timed on a
bounded sample of the same workload on this host's cores.
"""

from __future__ import annotations

import argparse
import json
import os
import sys
import time

ROOT = os.path.dirname(os.path.abspath(__file__))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)

import numpy as np  # noqa: E402

import synth  # noqa: E402

DEFAULT_WORKLOAD = "chatglm6b_26blk_ragged_32x1_recompute"
PEAK_TFLOPS = {"bf16": 2500.0, "f32": 157.3}   # dense matrix-core peaks, MI355X
PEAK_HBM_GBS = 8000.0
METRIC = "server-stack fwd+bwd tokens/sec and MFMA util %, ChatGLM-6B shape"
MFMA_CLASSES = ("gemm_nt_bias", "gemm_nt_bias_res", "gemm_nt_bias_gelu", "gemm_tn_acc", "gemm_nn_gelu_bwd",
                "gemm_nn", "attn_fwd", "attn_bwd", "lm_head_fwd", "lm_head_bwd")
GEMM_CLASSES = MFMA_CLASSES[:6]   # the block GEMMs
# Fragments of the kernel names rocprofv3 prints for each launch class of the
# bf16 path: the kernels that start an engine launch, then its later parts.
# CLASS_SOURCES: what they are built from (a stored counter reading is stale
# once their code, comments aside, changes).
CLASS_KERNELS = {
    # (layout, layout, epilogue; the tile shape follows.  One product may take
    # two launches on different tiles, and reduction slices: _classes)
    "gemm_nt_bias": (("gemm_bf16_kernel<true, true, 1,",), ()),
    "gemm_nt_bias_res": (("gemm_bf16_kernel<true, true, 2,",), ()),
    "gemm_nt_bias_gelu": (("gemm_bf16_kernel<true, true, 3,",), ()),
    "gemm_nn_gelu_bwd": (("gemm_bf16_kernel<true, false, 4,",), ()),
    "gemm_nn": (("gemm_bf16_kernel<true, false, 0,", "gemm_bf16_kernel<true, false, 6,"), ()),
    "gemm_tn_acc": (("gemm_bf16_kernel<false, false",), ("gemm_tile_slices_kernel",)),
    # few rows: a layer's input, weight and bias gradients in one launch (the
    # engine's launch timing shares it out among their classes)
    "gemm_pair": (("gemm_pair_kernel<",), ()),
    "attn_fwd": (("::fwd_kernel<",), ()),
    "attn_bwd": (("attn_delta_kernel",), ("::dkdv_kernel<", "::dq_kernel<", "::dq_ds_kernel<")),
    "layernorm_fwd": (("ln_fwd_kernel", "ln_fwd_row_kernel"), ()),
    "layernorm_bwd": (("ln_bwd_fused_kernel", "ln_bwd_dx_kernel"), ()),
    "rope_qk": (("rope_qk_kernel",), ()),
    "colsum": (("colsum_partial_kernel", "colsum_direct_kernel"), ("colsum_finish_kernel",)),
    "prefix_grad": (("prefix_grad_reduce_kernel",), ()),
    "adam": (("adam_kernel",), ()),
    "average": (("average_kernel",), ()),
}
# The fp32 sums of a token-major product's reduction slices (epilogue 7) belong
# to the class whose epilogue the kernel that adds them runs.
SLICED_KERNELS = {"gemm_bf16_kernel<true, true, 7,": {1: "gemm_nt_bias", 2: "gemm_nt_bias_res", 3: "gemm_nt_bias_gelu"},
                  "gemm_bf16_kernel<true, false, 7,": {0: "gemm_nn", 4: "gemm_nn_gelu_bwd", 6: "gemm_nn"}}
SLICE_SUM_KERNEL = "gemm_slices_kernel<"
CSRC = os.path.join(ROOT, "paper_2406_14898_amd", "csrc")
CLASS_SOURCES = {"gemm": ("gemm_bf16.hip", "common.h", "kernels.h"),
                 "attn": ("attention_bf16.hip", "attention.hip", "common.h", "kernels.h"),
                 "adam": ("optim.hip", "common.h"),
                 "average": ("optim.hip", "common.h"),
                 "": ("elementwise.hip", "common.h", "kernels.h")}
COPY_KERNEL = "neg_kernel"   # calibration: y = -x over float32, reads and writes the same bytes
# The paper's own efficiency figures (Section 4.1, the table comparing the
# training strategies' training time), quoted beside the measurement as
# context: end-to-end wall times of whole training runs on other hardware,
# with no token rate, so nothing here converts to this metric.
PAPER_CONTEXT = {
    "source": "Section 4.1, training time of the training strategies",
    "hardware": "NVIDIA A100 40 GB for the server and for each client",
    "workload": "1000 ReCoRD training points, P-tuning v2, batch 1 per client; sequence lengths not stated",
    "unit": "s (end-to-end wall time: client and server compute plus messaging)",
    "training_time_s": {"centralized": 166.4, "serial_2_clients": 175.2, "client_batch_2": 85.3,
                        "client_batch_4": 43.0, "client_batch_8": 22.5, "server_hierarchical_2": 87.3,
                        "server_hierarchical_3": 65.5, "server_hierarchical_5": 34.5,
                        "server_hierarchical_10": 17.3},
}


# String literals (kept: inline assembly lives in them), then // and /* */
# comments (dropped), for hashing the code the compiler sees.
_C_TOKENS = None


def code_text(src: str) -> str:
    """C/C++ source with comments removed and every run of whitespace made one
    space, so that editing a comment leaves the hash of the code unchanged."""
    import re
    global _C_TOKENS
    if _C_TOKENS is None:
        _C_TOKENS = re.compile(r'"(?:\\.|[^"\\\n])*"|//[^\n]*|/\*.*?\*/', re.S)
    kept = _C_TOKENS.sub(lambda m: m.group(0) if m.group(0).startswith('"') else " ", src)
    return " ".join(kept.split())


def class_source_hash(cls: str) -> str:
    import hashlib
    files = next(v for k, v in CLASS_SOURCES.items() if cls.startswith(k))
    h = hashlib.sha256()
    for f in files:
        with open(os.path.join(CSRC, f), encoding="utf-8") as fh:
            h.update(code_text(fh.read()).encode())
        h.update(b"\0")
    return h.hexdigest()[:16]


def traffic_file(workload: str) -> str:
    return os.path.join(ROOT, "profiles", f"server_stack_kernels_{workload}_hbm_traffic.txt")


def committed_traffic(cls: str, workload: str):
    """HBM bytes per launch of a class from the committed counter summary, or
    None if there is none or the kernel sources changed since it was taken."""
    path = traffic_file(workload)
    if not os.path.exists(path):
        return None
    for line in open(path):
        f = line.split()
        if len(f) >= 4 and f[0] == "class" and f[1] == cls:
            kv = dict(zip(f[2::2], f[3::2]))
            if kv.get("src") != class_source_hash(cls):
                return None
            return int(float(kv["hbm_bytes_per_launch"]))
    return None


PUBLISHED_SCLK_MHZ = 2400.0   # the clock the published matrix-core peaks assume


def sclk_path():
    """The amdgpu driver's shader-clock readout (pp_dpm_sclk) of device 0, or
    None where it is not readable."""
    import glob
    paths = sorted(glob.glob("/sys/class/drm/card*/device/pp_dpm_sclk"))
    if len(paths) == 1:
        return paths[0]
    try:
        import torch
        pr = torch.cuda.get_device_properties(0)
        bus = "%04x:%02x:%02x.0" % (pr.pci_domain_id, pr.pci_bus_id, pr.pci_device_id)
        for q in paths:
            if os.path.basename(os.path.realpath(os.path.dirname(q))) == bus:
                return q
    except Exception:
        pass
    return None


class ClockSampler:
    """Mean shader clock over a window: the current level of pp_dpm_sclk (the
    line marked '*'), read every 20 ms from a thread while the GPU runs."""

    def __init__(self, path):
        import threading
        self.path, self.samples, self._stop = path, [], threading.Event()
        self._t = threading.Thread(target=self._run, daemon=True) if path else None

    def _read(self):
        import re
        try:
            with open(self.path) as fh:
                m = re.search(r"(\d+)\s*Mhz\s*\*", fh.read(), re.IGNORECASE)
            return float(m.group(1)) if m else None
        except OSError:
            return None

    def _run(self):
        while not self._stop.is_set():
            v = self._read()
            if v is not None:
                self.samples.append(v)
            self._stop.wait(0.02)

    def start(self):
        if self._t:
            self._t.start()
        return self

    def stop(self):
        if self._t:
            self._stop.set()
            self._t.join()
        return (sum(self.samples) / len(self.samples)) if self.samples else None


def _short_kernel(name: str) -> str:
    name = (name[5:] if name.startswith("void ") else name).replace("flglm::(anonymous namespace)::", "")
    depth = 0
    for i, ch in enumerate(name):
        if ch == "<":
            depth += 1
        elif ch == ">":
            depth -= 1
        elif ch == "(" and depth == 0 and i > 0 and name[i - 1] != ":":
            return name[:i]
    return name


def _pmc_dispatches(d: str, counter: str, with_duration: bool = False) -> list:
    """[(queue, dispatch id, kernel name, counter value[, duration ns])] in
    dispatch order from a rocprofv3 --pmc CSV run."""
    import csv
    import glob
    out = []
    for f in glob.glob(os.path.join(d, "**", "*counter_collection.csv"), recursive=True):
        for r in csv.DictReader(open(f)):
            if r["Counter_Name"] == counter:
                row = (r["Queue_Id"], int(r["Dispatch_Id"]), r["Kernel_Name"], float(r["Counter_Value"]))
                if with_duration:
                    row += (float(r["End_Timestamp"]) - float(r["Start_Timestamp"]),)
                out.append(row)
    out.sort(key=lambda x: (x[0], x[1]))
    return out


def _class_of(name: str):
    """(class, starts a launch) of a kernel name, or (None, False).  A class's
    starting kernels begin an engine launch; its others are later parts of the
    same launch (the attention backward's three kernels, a column sum's
    finish)."""
    for cls, (starts, parts) in CLASS_KERNELS.items():
        if any(p in name for p in starts):
            return cls, True
        if any(p in name for p in parts):
            return cls, False
    return None, False


def _classes(dispatches) -> list:
    """_class_of every (queue, id, name, ...) dispatch in order.  A product in
    reduction slices is two dispatches in a row on its queue, the slices and
    their sum; the sum tells the class (a joint launch's sum follows it)."""
    out = [_class_of(d[2]) for d in dispatches]
    open_at = {}  # queue: index of the dispatch right before
    for i, d in enumerate(dispatches):
        q, name = d[0], d[2]
        j = open_at.get(q)
        if SLICE_SUM_KERNEL in name and j is not None:
            epi = int(name.split(SLICE_SUM_KERNEL)[1].split(">")[0])
            for pat, by_epi in SLICED_KERNELS.items():
                if pat in dispatches[j][2]:
                    out[j] = out[i] = (by_epi.get(epi), True)
            if out[j][0] == "gemm_pair":
                out[i] = ("gemm_pair", False)
        open_at[q] = i
    return out


def _class_launches(dispatches) -> dict:
    """{class: [engine launches, value total]} from (queue, id, name, value)
    dispatches in order.  A dispatch of the same kernel as the one right
    before it on its queue belongs to the same engine launch (the next piece
    of a GEMM cut along its reduction), and so does a GEMM dispatch of the same
    class (its rows past whole rounds on another tile, its reduction slices and
    their sum): the engine never runs two products of one class in a row.  A
    class's later kernel continues the launch its first kernel began, unless
    another class ran in between (a column-sum finish whose partial sums a GEMM
    epilogue produced is a launch of its own)."""
    out = {}
    prev, prev_cls = {}, {}
    for d, (cls, first) in zip(dispatches, _classes(dispatches)):
        q, name, v = d[0], d[2], d[3]
        if cls is not None:
            e = out.setdefault(cls, [0, 0.0])
            e[1] += v
            same = prev_cls.get(q) == cls
            if not (same and cls in GEMM_CLASSES) and prev.get(q) != name and (first or not same):
                e[0] += 1
        prev[q], prev_cls[q] = name, cls
    return out


def summarize_traffic(root: str, copy_mib: int, workload: str) -> str:
    """Text summary of four rocprofv3 --pmc runs under root: fetch/ and write/
    (FETCH_SIZE, WRITE_SIZE of the benchmark), copy_fetch/ and copy_write/ (the
    same counters for --copy-calibration).  Counter KiB are scaled by the
    ratio of the copy's known bytes to what the counter reads for it; per
    class also the average launch duration in the FETCH_SIZE run (dispatch
    timestamps) and the HBM rate the counters give over it."""
    copy_bytes = copy_mib << 20
    lines = []
    scale = {}
    for c, sub in (("FETCH_SIZE", "fetch"), ("WRITE_SIZE", "write")):
        hits = [v for _, _, k, v in _pmc_dispatches(os.path.join(root, "copy_" + sub), c) if COPY_KERNEL in k]
        n, v = len(hits), sum(hits)
        per = v / max(n, 1) * 1024.0
        scale[c] = copy_bytes / per
        lines.append(f"calibration {c} copy_bytes {copy_bytes} dispatches {n} counter_bytes_per_dispatch "
                     f"{per:.0f} factor {scale[c]:.4f}")
    fdisp = _pmc_dispatches(os.path.join(root, "fetch"), "FETCH_SIZE", with_duration=True)
    fetch = _class_launches(fdisp)
    write = _class_launches(_pmc_dispatches(os.path.join(root, "write"), "WRITE_SIZE"))
    # duration of each class's launches in the FETCH_SIZE run (dispatch timestamps)
    dur = _class_launches([(q, i, name, d) for q, i, name, _, d in fdisp])
    for cls in CLASS_KERNELS:
        n, fv = fetch.get(cls, (0, 0.0))
        n2, wv = write.get(cls, (0, 0.0))
        if n == 0:
            continue
        fb = fv / n * 1024.0 * scale["FETCH_SIZE"]
        wb = wv / max(n2, 1) * 1024.0 * scale["WRITE_SIZE"]
        us = dur.get(cls, (n, 0.0))[1] / n / 1e3
        gbs = (fb + wb) / (us * 1e-6) / 1e9 if us > 0 else 0.0
        lines.append(f"class {cls} launches {n} fetch_bytes_per_launch {fb:.0f} write_bytes_per_launch {wb:.0f} "
                     f"hbm_bytes_per_launch {fb + wb:.0f} avg_us {us:.1f} counter_gbs {gbs:.0f} "
                     f"src {class_source_hash(cls)}")
    return "\n".join(lines)


def summarize_mfma(root: str, bench_json: str = "") -> str:
    """Per class from one rocprofv3 --pmc "MfmaFlopsBF16 MfmaUtil" run under
    root: MFMA flops per engine launch as the hardware counts them (bf16 MFMA
    ops x 512), the same per launch from the engine's algorithmic count (the
    bench line in bench_json, when given), and the matrix cores' busy share
    while the class ran (MfmaUtil, weighted by dispatch duration)."""
    fl = _class_launches(_pmc_dispatches(root, "MfmaFlopsBF16"))
    util = {}
    busy = _pmc_dispatches(root, "MfmaUtil", with_duration=True)
    for (_, _, _, v, dur), (cls, _) in zip(busy, _classes(busy)):
        if cls is not None:
            e = util.setdefault(cls, [0.0, 0.0])
            e[0] += v * dur
            e[1] += dur
    alg = {}
    if bench_json:
        d = json.loads([l for l in open(bench_json) if l.startswith("{")][-1])
        for k, v in d["kernels"].items():
            if "tflops" in v:
                alg[k] = v["tflops"] * 1e12 * v["avg_launch_us"] * 1e-6
    out = [f"{'class':<20} {'launches':>8} {'counter_flop_per_launch':>24} {'algorithmic_flop_per_launch':>28} "
           f"{'ratio':>7} {'mfma_busy_pct':>14}"]
    for cls in CLASS_KERNELS:
        if cls not in fl or fl[cls][1] == 0:
            continue
        n, v = fl[cls]
        per = v / max(n, 1)
        a = alg.get(cls)
        u = util.get(cls)
        out.append(f"{cls:<20} {n:>8} {per:>24.4e} " + (f"{a:>28.4e} {per / a:>7.4f}" if a else f"{'-':>28} {'-':>7}") +
                   (f" {u[0] / u[1]:>14.1f}" if u and u[1] > 0 else f" {'-':>14}"))
    return "\n".join(out)


def summarize_trace(root: str) -> str:
    """Per-kernel table from a rocprofv3 --kernel-trace --stats CSV run, then
    per class the engine launches (grouped as in _class_launches) and their
    average duration."""
    import csv
    import glob
    rows = []
    for f in glob.glob(os.path.join(root, "**", "*kernel_stats.csv"), recursive=True):
        rows += list(csv.DictReader(open(f)))
    rows.sort(key=lambda r: -float(r["TotalDurationNs"]))
    out = [f"{'kernel':<72} {'calls':>6} {'avg_us':>10} {'total_ms':>10} {'pct':>6}"]
    for r in rows:
        out.append(f"{_short_kernel(r['Name'])[:72]:<72} {int(r['Calls']):>6} {float(r['AverageNs']) / 1e3:>10.1f} "
                   f"{float(r['TotalDurationNs']) / 1e6:>10.2f} {float(r['Percentage']):>6.2f}")
    disp = []
    for f in glob.glob(os.path.join(root, "**", "*kernel_trace.csv"), recursive=True):
        for r in csv.DictReader(open(f)):
            disp.append((r["Queue_Id"], int(r["Dispatch_Id"]), r["Kernel_Name"],
                         float(r["End_Timestamp"]) - float(r["Start_Timestamp"])))
    disp.sort(key=lambda x: (x[0], x[1]))
    by_cls = _class_launches(disp)
    out.append("")
    out.append(f"{'class':<20} {'launches':>8} {'avg_us_per_launch':>18}")
    for cls, (n, t) in sorted(by_cls.items(), key=lambda kv: -kv[1][1]):
        out.append(f"{cls:<20} {n:>8} {t / max(n, 1) / 1e3:>18.1f}")
    return "\n".join(out)


def copy_calibration(mib: int) -> None:
    """A plain streaming kernel of known size for scaling the HBM counters:
    y = -x over mib MiB of float32 (reads and writes mib MiB each), 3 times."""
    import torch
    n = (mib << 20) // 4
    x = torch.ones(n, device="cuda", dtype=torch.float32)
    y = torch.empty_like(x)
    for _ in range(3):
        torch.neg(x, out=y)
    torch.cuda.synchronize()
    print(json.dumps({"copy_calibration_bytes": mib << 20, "dispatches": 3}))


def total_layers(w: synth.Workload) -> int:
    """Blocks a step runs: the server's, plus the client's blocks 0 and N-1
    for the whole split model."""
    return w.shape.num_layers + (2 if w.vocab else 0)


# Stored softmax-gradient cap of the engine's backward (above it, dq
# recomputes S and dP).
ATTN_DS_MAX_BYTES = 8 << 30


def attn_ds_stored(w, b, F):
    """Whether the engine's attention backward stores dS for this batch."""
    if not w.backward or w.dtype != "bf16":
        return False
    prefix = b.prefix_len if w.mask == "prefix" else None
    return F.fl_test_attention_ds_bytes(b.cu_seqlens, prefix, w.shape.num_heads, w.num_prefix) <= ATTN_DS_MAX_BYTES


def vocab_padded(w: synth.Workload) -> int:
    return (w.vocab + 255) // 256 * 256


def algorithmic_flops(w: synth.Workload, b: synth.Batch) -> dict:
    """Per step: GEMM 8 H^2 + 4 H F per token per block forward (24 H^2 at
    F = 4 H), twice that backward (once with frozen weights: input gradients
    only); attention 4 H per
    visible (query, key) pair forward, 8 H backward, a P-tuning v2 prefix
    adding L_p pairs per token.  The whole split model adds the final
    linear layer: 2 V H per token forward, 2 V H backward for the input
    gradient and 2 V H for the weight gradient unless frozen.
    Recomputation is not counted."""
    H = w.shape.hidden
    T = b.total_tokens
    pairs = float(w.num_prefix) * T
    for s in range(b.num_seqs):
        L = float(b.seqlens[s])
        P = float(b.prefix_len[s]) if b.mask == "prefix" else 0.0
        pairs += L * (L + 1) / 2 + (P * (P - 1) / 2 if P > 1 else 0.0)
    F = w.shape.ffn_hidden
    fwd_g = 8.0 * H * H + 4.0 * H * F   # QKV 6 H^2, out-projection 2 H^2, FFN 4 H F
    mult_g = ((2 if w.frozen else 3) if w.backward else 1) * fwd_g
    mult_a = 12 if w.backward else 4
    g = mult_g * T * total_layers(w)
    a = mult_a * H * pairs * total_layers(w)
    head = (2.0 + 2.0 + (0.0 if w.frozen else 2.0)) * w.vocab * H * T if w.vocab else 0.0
    return {"gemm": g, "attention": a, "lm_head": head, "total": g + a + head, "pairs": pairs}


def trained_shapes(w: synth.Workload):
    """(name, shape) of every trained tensor, layer-major: the P-tuning v2
    prefixes when the weights are frozen, else every weight and bias."""
    out = []
    for l in range(total_layers(w)):
        if w.frozen:
            out += [(f"{l}.{k}", (w.num_prefix, w.shape.hidden)) for k in ("prefix_k", "prefix_v")]
        else:
            out += [(f"{l}.{k}", s) for k, s in synth.param_shapes(w.shape).items()]
            out += [(f"{l}.{k}", (w.num_prefix, w.shape.hidden)) for k in ("prefix_k", "prefix_v")[
                :2 if w.num_prefix else 0]]
    if w.vocab and not w.frozen:
        out += [("embedding", (w.vocab, w.shape.hidden)), ("lm_head", (w.vocab, w.shape.hidden))]
    return out


def device_inputs(w: synth.Workload, b: synth.Batch, seed: int, arena: bool = False):
    """Seeded device-side draws (torch Philox on the GPU) with the workload's
    distributions: weights and biases N(0, 0.02), LayerNorm gains 1 + N(0, 0.02),
    x ~ N(0, 1), dy ~ N(0, dy_std); rounded to bf16 for bf16 workloads.
    arena: the trained tensors live in one ParamArena (fp32 masters holding
    the draws, fp32 gradients and Adam moments, bf16 compute copy); the stack
    reads and accumulates into views of it.  The whole split model adds the
    client's blocks (layers 0 and N-1 around the server's), an embedding
    table ~ N(0, 1) (so block 0 sees activations of the server's scale) and
    a final linear layer ~ N(0, 0.02).  Returns a dict: layers, grads, x, dy,
    arena (or None), embedding, lm_head and their gradients (None: frozen)."""
    import torch

    from paper_2406_14898_amd import ParamArena
    dt = torch.bfloat16 if w.dtype == "bf16" else torch.float32
    shapes = synth.param_shapes(w.shape)
    gen = torch.Generator(device="cuda")
    ar = ParamArena(trained_shapes(w), bf16_copy=w.dtype == "bf16") if arena else None
    mv = ar.master_views() if ar else {}
    params, grads = [], []
    for l in range(total_layers(w)):
        gen.manual_seed(seed * 100003 + l)
        draws = {}
        for name, shp in shapes.items():
            t = torch.randn(shp, generator=gen, device="cuda", dtype=torch.float32) * 0.02
            if name in ("ln1_g", "ln2_g"):
                t += 1.0
            draws[name] = t
        for name in ("prefix_k", "prefix_v")[:2 if w.num_prefix else 0]:  # P-tuning v2 prefix ~ N(0, 1)
            draws[name] = torch.randn((w.num_prefix, w.shape.hidden), generator=gen, device="cuda")
        p = {}
        for name, t in draws.items():
            if f"{l}.{name}" in mv:
                mv[f"{l}.{name}"].copy_(t)
            else:
                p[name] = t.to(dt)
        del draws
        params.append(p)
        grads.append({k: torch.zeros(v.shape, dtype=torch.float32, device="cuda") for k, v in p.items()
                      if not w.frozen or k.startswith("prefix_")})
    out = {"embedding": None, "lm_head": None, "g_embedding": None, "g_lm_head": None}
    if w.vocab:
        gen.manual_seed(seed * 100003 + 99989)
        for name, std in (("embedding", 1.0), ("lm_head", 0.02)):
            t = torch.randn((w.vocab, w.shape.hidden), generator=gen, device="cuda") * std
            if name in mv:
                mv[name].copy_(t)
            else:
                out[name] = t.to(dt)
            del t
    if ar:
        ar.refresh_compute()
        cv, gv = ar.compute_views(), ar.grad_views()
        for key in ar.names:
            if "." not in key:
                out[key], out["g_" + key] = cv[key], gv[key]
                continue
            l, name = key.split(".", 1)
            params[int(l)][name] = cv[key]
            grads[int(l)][name] = gv[key]
    elif w.vocab and not w.frozen:
        out["g_embedding"] = torch.zeros((w.vocab, w.shape.hidden), dtype=torch.float32, device="cuda")
        out["g_lm_head"] = torch.zeros((w.vocab, w.shape.hidden), dtype=torch.float32, device="cuda")
    gen.manual_seed(seed * 100003 + 99991)
    T, H = b.total_tokens, w.shape.hidden
    out["x"] = out["dy"] = None
    if not w.vocab:
        out["x"] = torch.randn((T, H), generator=gen, device="cuda", dtype=torch.float32).to(dt)
        out["dy"] = (torch.randn((T, H), generator=gen, device="cuda", dtype=torch.float32) * w.dy_std).to(dt)
    out.update(layers=params, grads=grads, arena=ar)
    return out


def average_bench(w: synth.Workload, replicas: int, launches: int) -> dict:
    """Times the server-hierarchical aggregation alone: the mean of
    `replicas` copies of the workload's trained parameters (fp32, with bf16
    compute copies for bf16 workloads), written back to every replica."""
    import torch

    from paper_2406_14898_amd import flglm as F
    n = sum(int(np.prod(s)) for _, s in trained_shapes(w))
    per = 4 + 4 + (2 if w.dtype == "bf16" else 0)   # read fp32, write fp32 (+ bf16) per replica and element
    if replicas * n * (6 if w.dtype == "bf16" else 4) > 200e9:
        raise SystemExit(f"{replicas} replicas of {n} parameters do not fit beside the allocator's headroom")
    gen = torch.Generator(device="cuda").manual_seed(0)
    reps = [torch.randn(n, generator=gen, device="cuda") for _ in range(replicas)]
    c16 = [torch.empty(n, dtype=torch.bfloat16, device="cuda") for _ in range(replicas)] \
        if w.dtype == "bf16" else None
    stream = torch.cuda.current_stream()
    F.fl_average_replicas(reps, c16, n, stream)
    ev = [torch.cuda.Event(enable_timing=True) for _ in range(launches + 1)]
    torch.cuda.synchronize()
    ev[0].record(stream)
    for i in range(launches):
        F.fl_average_replicas(reps, c16, n, stream)
        ev[i + 1].record(stream)
    torch.cuda.synchronize()
    us = ev[0].elapsed_time(ev[-1]) / launches * 1e3
    nbytes = replicas * n * per
    gbs = nbytes / (us / 1e6) / 1e9
    return {"metric": "server-hierarchical replica averaging (one launch)", "kernel": "average",
            "workload": w.name, "replicas": replicas, "params": n, "launches": launches,
            "avg_launch_us": round(us, 2), "bytes_per_launch": nbytes, "achieved_gbs": round(gbs, 1),
            "peak": PEAK_HBM_GBS, "unit": "GB/s", "frac": round(gbs / PEAK_HBM_GBS, 4)}


def spread_order(lengths) -> list:
    """Sequence indices in an order whose every prefix spreads over the
    length distribution: the sequences at the quantiles 1/2, 1/4, 3/4, 1/8,
    3/8, ... of the sorted lengths (van der Corput order), each once."""
    order = list(np.argsort(np.asarray(lengths), kind="stable"))
    n, out, seen = len(order), [], set()
    k = 1
    while len(out) < n:
        den = 1 << k.bit_length()
        i = int((int(f"{k:b}"[::-1], 2) / den) * n) if k > 0 else 0
        k += 1
        for j in (i, *range(n)):  # nearest not yet taken, upwards then from the start
            if j < n and order[j] not in seen:
                seen.add(order[j])
                out.append(int(order[j]))
                break
    return out


def cpu_baseline(w: synth.Workload, b: synth.Batch, budget_s: float) -> dict:
    """The CPU oracle (float32, numpy BLAS) on a bounded sample: one block's
    forward + recompute + backward over whole sequences of the workload, taken
    in an order that spreads over its length distribution (``spread_order``),
    until the budget is used; scaled to the full stack depth."""
    import oracle
    blas = "unknown"
    try:
        from threadpoolctl import threadpool_info
        info = [i for i in threadpool_info() if i.get("user_api") == "blas"]
        threads = max((i.get("num_threads", 1) for i in info), default=1)
        if info:
            blas = f"{info[0].get('internal_api')} {info[0].get('version')}"
    except Exception:  # pragma: no cover
        threads = len(os.sched_getaffinity(0))
    cpu = "unknown"
    try:
        with open("/proc/cpuinfo") as f:
            cpu = next((l.split(":", 1)[1].strip() for l in f if l.startswith("model name")), "unknown")
    except OSError:  # pragma: no cover
        pass
    one = synth.StackShape(1, w.shape.hidden, w.shape.num_heads, w.shape.ffn_hidden, w.shape.rotary_dim,
                           w.shape.rope_base, w.shape.ln_eps)
    layer = synth.layer_params(w.shape, 0, seed=0, bf16=w.dtype == "bf16")
    if w.num_prefix:
        layer.update(synth.prefix_params(w.shape, 0, w.num_prefix, seed=0, bf16=w.dtype == "bf16"))
    f32 = np.float32
    grads = ([oracle.zero_prefix_grads(w.num_prefix, w.shape.hidden, f32)] if w.frozen
             else [oracle.zero_grads(one, f32)])
    done_tokens, spent = 0, 0.0
    seqs = []
    for s in spread_order(b.seqlens):
        sub = synth.Batch(np.array([0, int(b.seqlens[s])], np.int32), np.array([0, 1], np.int32), b.mask,
                          None if b.prefix_len is None else np.array([int(b.prefix_len[s])], np.int32))
        L = sub.total_tokens
        x = synth.activations(L, w.shape.hidden, seed=1, bf16=w.dtype == "bf16")
        dy = synth.upstream_grad(L, w.shape.hidden, seed=1, bf16=w.dtype == "bf16", std=w.dy_std)
        t0 = time.perf_counter()
        y, xs = oracle.stack_forward([layer], 1, x, sub, one, f32)
        if w.backward:
            oracle.stack_backward([layer], 1, xs, dy, sub, one, grads, f32)
        spent += time.perf_counter() - t0
        done_tokens += L
        seqs.append(L)
        if spent >= budget_s:
            break
    per_block_tok_s = done_tokens / spent
    nl = total_layers(w)
    sec_per_tok = nl / per_block_tok_s
    head = ""
    if w.vocab:
        # the final linear layer with the loss, forward and backward, on a few tokens
        n = 32
        g = np.random.default_rng(3)
        wv = (g.standard_normal((w.vocab, w.shape.hidden)) * 0.02).astype(f32)
        h = g.standard_normal((n, w.shape.hidden)).astype(f32)
        lab = g.integers(0, w.vocab, n)
        t0 = time.perf_counter()
        lg, lse, _, _ = oracle.client.lm_head_forward(h, wv, lab)
        oracle.client.lm_head_backward(h, wv, lg, lse, lab, 1.0 / n)
        th = time.perf_counter() - t0
        del wv, lg
        sec_per_tok += th / n
        head = f"; final linear layer + loss (vocab {w.vocab}) fwd+bwd on {n} tokens in {th:.1f} s"
    return {
        "value": 1.0 / sec_per_tok,
        "unit": "tokens/s",
        "cores": int(threads),
        "kind": "oracle",
        "sample": (f"1 of {nl} blocks, {'fwd+recompute+bwd' if w.backward else 'fwd'}, float32, "
                   f"{len(seqs)} whole sequence(s) spread over the workload's length distribution "
                   f"(lengths {seqs}, workload {int(b.seqlens.min())}..{int(b.seqlens.max())}, "
                   f"mean {float(b.seqlens.mean()):.0f}; {done_tokens} tokens) in {spent:.1f} s; "
                   f"per-token time times {nl} blocks{head}; host {cpu}, BLAS {blas}, "
                   f"{len(os.sched_getaffinity(0))} cores visible"),
    }


SECONDARY_WORKLOADS = (
    ("chatglm6b_1blk_fwd_4x4x512", 10, 3),
    ("chatglm6b_1blk_ragged_8x4", 10, 3),
    ("chatglm6b_26blk_prefix_16x2x512", 3, 1),
    ("chatglm6b_26blk_ptuning128_ragged_32x1_recompute", 3, 1),
)


def secondary_run(name: str, seed: int, steps: int, warmup: int) -> dict:
    """A short timed run of another server-stack workload (same device
    draws): tokens/s, ms per step, algorithmic MFMA utilisation and the
    GEMMs' MFMA utilisation (their launch times from one more, untimed step
    with launch timing on)."""
    import torch

    from paper_2406_14898_amd import BatchDesc, ServerStack
    from paper_2406_14898_amd import flglm as F
    w = synth.WORKLOADS[name]
    b = w.batch(seed=seed)
    sh = w.shape
    inp = device_inputs(w, b, seed)
    params, grads, x, dy = inp["layers"], inp["grads"], inp["x"], inp["dy"]
    ss = ServerStack(sh.num_layers, sh.hidden, sh.num_heads, sh.ffn_hidden, sh.rotary_dim, w.dtype, sh.rope_base,
                     sh.ln_eps, w.num_prefix)
    bd = BatchDesc.from_batch(b)
    saved, ws = ss.buffers(bd, w.recompute, with_saved=w.backward)
    y = torch.empty_like(x)
    dx = torch.empty_like(x) if w.backward else None
    stream = torch.cuda.current_stream()

    def step():
        ss.forward(bd, params, x, y, saved, ws, w.recompute, stream)
        if w.backward:
            ss.backward(bd, params, grads, x, saved, dy, dx, ws, w.recompute, stream)

    for _ in range(warmup):
        step()
    torch.cuda.synchronize()
    # launch timing in one untimed step (the GEMM classes' times), then the
    # timed steps without events
    F.fl_stack_profile(ss.handle, 1)
    step()
    torch.cuda.synchronize()
    prof = F.profile_table(ss.handle)
    F.fl_stack_profile(ss.handle, 0)
    e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    e0.record(stream)
    for _ in range(steps):
        step()
    e1.record(stream)
    torch.cuda.synchronize()
    ms = e0.elapsed_time(e1) / steps
    ss.close()
    del inp, params, grads, x, dy, y, dx, saved, ws
    torch.cuda.empty_cache()
    peak = PEAK_TFLOPS[w.dtype] * 1e12
    gemm_ms = sum(prof[k]["ms"] for k in GEMM_CLASSES if k in prof)
    gemm_fl = sum(prof[k]["flops"] for k in GEMM_CLASSES if k in prof)
    fl = algorithmic_flops(w, b)
    return {"tokens_s": round(b.total_tokens / (ms / 1e3), 1), "ms_per_step": round(ms, 3), "steps": steps,
            "warmup": warmup, "total_tokens": b.total_tokens, "blocks": sh.num_layers,
            "backward": w.backward, "recompute": w.recompute, "mask": w.mask, "ptuning_prefix": w.num_prefix,
            "mfma_util": round(fl["total"] / (ms / 1e3) / peak, 4),
            "gemm_mfma_util": round(gemm_fl / (gemm_ms / 1e3) / peak, 4) if gemm_ms else None}


def main() -> int:
    ap = argparse.ArgumentParser(description=__doc__.split("\n")[0])
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=5)
    ap.add_argument("--warmup", type=int, default=2)
    ap.add_argument("--workload", default=DEFAULT_WORKLOAD, choices=sorted(synth.WORKLOADS))
    ap.add_argument("--seed", type=int, default=0)
    ap.add_argument("--cpu-budget", type=float, default=15.0, help="seconds of CPU oracle work")
    ap.add_argument("--no-cpu-baseline", action="store_true")
    ap.add_argument("--no-secondary", action="store_true",
                    help="skip the short runs of the other workloads reported under 'secondary'")
    ap.add_argument("--no-profile", action="store_true", help="time without per-launch events")
    ap.add_argument("--copy-calibration", type=int, metavar="MIB",
                    help="only run the counter-calibration copy kernel over MIB MiB")
    ap.add_argument("--summarize-traffic", metavar="DIR",
                    help="print the HBM traffic summary of rocprofv3 --pmc runs under DIR (no GPU)")
    ap.add_argument("--summarize-mfma", metavar="DIR",
                    help="print MFMA counter summary of a rocprofv3 --pmc 'MfmaFlopsBF16 MfmaUtil' run")
    ap.add_argument("--bench-json", default="", help="bench line to compare --summarize-mfma with")
    ap.add_argument("--summarize-trace", metavar="DIR",
                    help="print the per-kernel table of a rocprofv3 --kernel-trace --stats run (no GPU)")
    ap.add_argument("--copy-mib", type=int, default=1024, help="size the calibration run used")
    ap.add_argument("--update", choices=("none", "adam"), default="none",
                    help="adam: each step ends with the Adam update of every trained parameter "
                         "(one launch over a flat arena; gradients cleared in the same pass)")
    ap.add_argument("--average-bench", type=int, metavar="M",
                    help="only time the averaging of M replicas of the workload's trained parameters")
    args = ap.parse_args()
    if args.summarize_traffic:
        print(summarize_traffic(args.summarize_traffic, args.copy_mib, args.workload))
        return 0
    if args.summarize_mfma:
        print(summarize_mfma(args.summarize_mfma, args.bench_json))
        return 0
    if args.summarize_trace:
        print(summarize_trace(args.summarize_trace))
        return 0
    if args.copy_calibration:
        copy_calibration(args.copy_calibration)
        return 0

    if args.gpus != 1 or int(os.environ.get("WORLD_SIZE", "1")) != 1:
        print(json.dumps({"error": "bench.py runs the server stack on one GPU only; "
                                   f"--gpus {args.gpus} is not supported (multi-GPU sharding is design-only)"}))
        return 2

    import torch

    from paper_2406_14898_amd import BatchDesc, ServerStack, SplitModel
    from paper_2406_14898_amd import flglm as F

    assert torch.cuda.is_available(), "bench.py needs a GPU"
    torch.cuda.set_device(0)
    w = synth.WORKLOADS[args.workload]
    b = w.batch(seed=args.seed)
    T = b.total_tokens
    print(f"[bench] workload {w.name}: T={T} S={b.num_seqs} C={b.num_clients} maxL={b.max_seqlen}", file=sys.stderr,
          flush=True)
    if args.average_bench:
        print(json.dumps(average_bench(w, args.average_bench, max(args.steps, 1))))
        return 0
    inp = device_inputs(w, b, args.seed, arena=args.update == "adam")
    arena = inp["arena"]
    if arena is not None and not w.backward:
        raise SystemExit("--update adam needs a workload with a backward pass")
    params, grads = inp["layers"], inp["grads"]
    sh = w.shape
    bd = BatchDesc.from_batch(b)
    stream = torch.cuda.current_stream()
    client_marks = []  # (class, start event, end event) of the client-side calls
    if w.vocab:
        # the whole split model: client embedding + block 0, the server's
        # blocks, client block N-1 + final linear layer and loss
        model = SplitModel(sh.hidden, sh.num_heads, sh.ffn_hidden, sh.rotary_dim, sh.num_layers, w.vocab, w.dtype,
                           sh.rope_base, sh.ln_eps, w.num_prefix, sh.residual_alpha, sh.rotary_2d)
        handles = [model.block0.handle, model.server.handle, model.block_last.handle]
        buf = model.buffers(bd, w.recompute)
        ids, labels = synth.token_ids(b, w.vocab, args.seed)
        scale = 1.0 / max(1, int((labels >= 0).sum()))
        sp = {"embedding": inp["embedding"], "lm_head": inp["lm_head"], "block0": params[0],
              "server": params[1:-1], "block_last": params[-1]}
        sg = {"embedding": inp["g_embedding"], "lm_head": inp["g_lm_head"], "block0": grads[0],
              "server": grads[1:-1], "block_last": grads[-1]}
        if sh.residual_alpha > 0:  # ChatGLM-6B's final LayerNorm: 1 + N(0, 0.02), N(0, 0.02)
            gen = torch.Generator(device="cuda").manual_seed(args.seed * 100003 + 99983)
            tdt = torch.bfloat16 if w.dtype == "bf16" else torch.float32
            sp["final_ln_g"] = (1 + 0.02 * torch.randn(sh.hidden, generator=gen, device="cuda")).to(tdt)
            sp["final_ln_b"] = (0.02 * torch.randn(sh.hidden, generator=gen, device="cuda")).to(tdt)
            if not w.frozen:
                sg["final_ln_g"] = torch.zeros(sh.hidden, device="cuda")
                sg["final_ln_b"] = torch.zeros(sh.hidden, device="cuda")

        def fwd_bwd(timed):
            model.step(bd, ids, labels, sp, sg, scale, buf, w.recompute, stream, client_marks if timed else None)
        close = model.close
    else:
        ss = ServerStack(sh.num_layers, sh.hidden, sh.num_heads, sh.ffn_hidden, sh.rotary_dim, w.dtype, sh.rope_base,
                         sh.ln_eps, w.num_prefix)
        handles = [ss.handle]
        saved, ws = ss.buffers(bd, w.recompute, with_saved=w.backward)
        x, dy = inp["x"], inp["dy"]
        y = torch.empty_like(x)
        dx = torch.empty_like(x) if w.backward else None

        def fwd_bwd(timed):
            ss.forward(bd, params, x, y, saved, ws, w.recompute, stream)
            if w.backward:
                ss.backward(bd, params, grads, x, saved, dy, dx, ws, w.recompute, stream)
        close = ss.close

    upd_events = []

    def step(marks=False):
        fwd_bwd(marks)
        if arena is not None:
            e = (torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True))
            e[0].record(stream)
            arena.adam_step(zero_grad=True, stream=stream)
            e[1].record(stream)
            upd_events.append(e)

    def collect():
        table = {}
        for h in handles:
            for k, r in F.profile_table(h).items():
                e = table.setdefault(k, dict(launches=0, ms=0.0, flops=0.0, bytes=0.0))
                for f in e:
                    e[f] += r[f]
        return table

    for i in range(args.warmup):
        step()
        torch.cuda.synchronize()
        print(f"[bench] warmup step {i + 1}/{args.warmup} done", file=sys.stderr, flush=True)
    # Per-class breakdown from one more (untimed) step with every launch
    # between two events; the timed steps then bracket only the dominant
    # class, whose live launch times give roofline.achieved (two events per
    # launch cost 0.3-0.5 % of a step when every launch carries them).
    prof, prof_steps, dom_mask = {}, 0, 0
    if not args.no_profile:
        for h in handles:
            F.fl_stack_profile(h, True)
        client_marks.clear()
        step(marks=True)
        torch.cuda.synchronize()
        prof, prof_steps = collect(), 1
        for h in handles:
            F.fl_stack_profile(h, False)
        if w.vocab:
            # client-side calls timed with events on the same stream
            H, Vp = sh.hidden, vocab_padded(w)
            work = {"lm_head_fwd": (2.0 * T * Vp * H, 0.0),
                    "lm_head_bwd": ((2.0 if w.frozen else 4.0) * T * Vp * H, 0.0),
                    "embedding_fwd": (0.0, 2.0 * T * H * (2 if w.dtype == "bf16" else 4)),
                    "embedding_bwd": (0.0, T * H * ((2 if w.dtype == "bf16" else 4) + 8.0))}
            for name, a, e in client_marks:
                r = prof.setdefault(name, dict(launches=0, ms=0.0, flops=0.0, bytes=0.0))
                r["launches"] += 1
                r["ms"] += a.elapsed_time(e)
                r["flops"] += work[name][0]
                r["bytes"] += work[name][1]
        engine_classes = {F.fl_profile_class_name(c): c for c in range(F.FL_PROF_NUM_CLASSES)}
        dom_engine = max((k for k in prof if k in engine_classes), key=lambda k: prof[k]["ms"], default=None)
        if dom_engine is not None:
            dom_mask = 1 << engine_classes[dom_engine]
        print(f"[bench] breakdown step done; timing {dom_engine} live", file=sys.stderr, flush=True)
    upd_events.clear()
    for h in handles:
        F.fl_stack_profile_classes(h, dom_mask)
    marks = [torch.cuda.Event(enable_timing=True) for _ in range(args.steps + 1)]
    torch.cuda.synchronize()
    clock = ClockSampler(sclk_path()).start()
    marks[0].record(stream)
    for i in range(args.steps):
        step()
        marks[i + 1].record(stream)
    torch.cuda.synchronize()
    sclk = clock.stop()
    ms = marks[0].elapsed_time(marks[-1]) / args.steps
    per_step = sorted(marks[i].elapsed_time(marks[i + 1]) for i in range(args.steps))
    live = collect() if dom_mask else {}
    for h in handles:
        F.fl_stack_profile(h, False)
    print(f"[bench] timed {args.steps} steps: {ms:.2f} ms/step", file=sys.stderr, flush=True)

    flops = algorithmic_flops(w, b)
    peak = PEAK_TFLOPS[w.dtype]
    tok_s = T / (ms / 1e3)
    kernels = {}
    for name, r in sorted(prof.items(), key=lambda kv: -kv[1]["ms"]):
        per_ms = r["ms"] / r["launches"]
        ent = {"launches": r["launches"], "ms_per_step": round(r["ms"] / prof_steps, 3),
               "avg_launch_us": round(per_ms * 1e3, 2)}
        if r["flops"] > 0:
            ent["tflops"] = round(r["flops"] / (r["ms"] / 1e3) / 1e12, 1)
        if r["bytes"] > 0 and name not in MFMA_CLASSES:
            ent["gbs"] = round(r["bytes"] / (r["ms"] / 1e3) / 1e9, 1)
        kernels[name] = ent
    # hardware flops: every launch's own count (forward recompute launches
    # included); the attention backward computes S and dP once and dq from the
    # stored dS (10 H per pair against the 8 H counted as algorithmic), or,
    # when that store would pass its cap, recomputes S and dP for dq (14 H)
    attn_hw = 10.0 / 8.0 if attn_ds_stored(w, b, F) else 14.0 / 8.0
    hw_flops = (sum(r["flops"] * (attn_hw if k == "attn_bwd" else 1.0) for k, r in prof.items()) / prof_steps
                if prof_steps else 0.0)
    gemm_ms = sum(prof[k]["ms"] for k in GEMM_CLASSES if k in prof)
    gemm_fl = sum(prof[k]["flops"] for k in GEMM_CLASSES if k in prof)
    roofline = None
    if prof:
        # the dominant class of the breakdown step, with its launches timed live
        # during the timed steps
        dom = max(live, key=lambda k: live[k]["ms"]) if live else max(prof, key=lambda k: prof[k]["ms"])
        r = live.get(dom, prof[dom])
        avg_s = r["ms"] / r["launches"] / 1e3
        if dom in MFMA_CLASSES:
            ach = r["flops"] / r["launches"] / avg_s / 1e12
            roofline = {"kernel": dom, "bound": "mfma", "achieved": round(ach, 1), "peak": peak, "unit": "TFLOP/s",
                        "frac": round(ach / peak, 4),
                        "traffic": committed_traffic(dom, w.name)}
        else:
            ach = r["bytes"] / r["launches"] / avg_s / 1e9
            roofline = {"kernel": dom, "bound": "hbm", "achieved": round(ach, 1), "peak": PEAK_HBM_GBS,
                        "unit": "GB/s", "frac": round(ach / PEAK_HBM_GBS, 4),
                        "traffic": committed_traffic(dom, w.name)}

    out = {
        "metric": METRIC,
        "value": round(tok_s, 1),
        "unit": "tokens/s",
        "n_gpus": 1,
        "steps": args.steps,
        "warmup": args.warmup,
        "ms_per_step": round(ms, 3),
        "higher_is_better": True,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": w.dtype,
        "data": ("synthetic (seeded device draws: weights N(0,0.02), %s%s)" % (
            "embedding N(0,1), token ids uniform over the vocabulary, next-token labels" if w.vocab else
            "x N(0,1), dy N(0,%g)" % w.dy_std, ", prefix keys/values N(0,1)" if w.num_prefix else "")),
        "config": {"workload": w.name, "clients": b.num_clients, "seqs": b.num_seqs, "total_tokens": T,
                   "max_seqlen": b.max_seqlen, "blocks": w.shape.num_layers, "hidden": w.shape.hidden,
                   "heads": w.shape.num_heads, "ffn": w.shape.ffn_hidden, "mask": w.mask,
                   "backward": w.backward, "recompute": w.recompute, "parallelism": "single GPU",
                   "ptuning_prefix": w.num_prefix, "weights_frozen": w.frozen,
                   "block": ("ChatGLM-6B (alpha %.3f residual, 2-D positions%s)" % (
                       w.shape.residual_alpha, ", final LayerNorm" if w.vocab else "")
                             if w.shape.residual_alpha else "pre-LN, x + f(LN(x)), 1-D positions"),
                   "scope": ("whole split model: client embedding + block 0, %d server blocks, client block %d + "
                             "final linear (vocab %d) + cross-entropy" % (w.shape.num_layers, w.shape.num_layers + 1,
                                                                          w.vocab)) if w.vocab else "server stack"},
        "ms_per_step_median": round(per_step[len(per_step) // 2], 3),
        "ms_per_step_min": round(per_step[0], 3),
        "mfma_util": round(flops["total"] / (ms / 1e3) / (peak * 1e12), 4),
        "hfu": round(hw_flops / (ms / 1e3) / (peak * 1e12), 4) if hw_flops else None,
        "hardware_tflop_per_step": round(hw_flops / 1e12, 3) if hw_flops else None,
        "gemm_mfma_util": round(gemm_fl / (gemm_ms / 1e3) / (peak * 1e12), 4) if gemm_ms else None,
        "algorithmic_tflop_per_step": round(flops["total"] / 1e12, 3),
        # the same utilisations against the peak at the shader clock measured
        # during the timed steps (the published peak assumes 2400 MHz)
        "sclk_mhz_mean": round(sclk, 1) if sclk else None,
        "mfma_util_at_clock": (round(flops["total"] / (ms / 1e3) / (peak * 1e12) * PUBLISHED_SCLK_MHZ / sclk, 4)
                               if sclk else None),
        "gemm_mfma_util_at_clock": (round(gemm_fl / (gemm_ms / 1e3) / (peak * 1e12) * PUBLISHED_SCLK_MHZ / sclk, 4)
                                    if sclk and gemm_ms else None),
        "roofline": roofline,
        "kernels": kernels,
        "cpu_baseline": None,
        "paper_context": PAPER_CONTEXT,
    }
    if arena is not None:
        # read p, g, m, v; write p, m, v, the bf16 copy and the cleared g
        per = 16 + 12 + 4 + (2 if arena.compute is not None else 0)
        us = sum(a.elapsed_time(c) for a, c in upd_events) / len(upd_events) * 1e3
        gbs = per * arena.n / (us / 1e6) / 1e9
        out["config"]["update"] = "adam"
        out["update"] = {"kernel": "adam", "params": arena.n, "launches": len(upd_events),
                         "avg_launch_us": round(us, 2), "bytes_per_launch": per * arena.n,
                         "achieved_gbs": round(gbs, 1), "peak": PEAK_HBM_GBS, "unit": "GB/s",
                         "frac": round(gbs / PEAK_HBM_GBS, 4)}
    close()
    del inp, params, grads
    torch.cuda.empty_cache()
    if not args.no_secondary and args.workload == DEFAULT_WORKLOAD and arena is None:
        out["secondary"] = {}
        for name, n_steps, n_warm in SECONDARY_WORKLOADS:
            try:
                out["secondary"][name] = secondary_run(name, args.seed, n_steps, n_warm)
            except Exception as e:  # pragma: no cover - reported, the headline line still prints
                out["secondary"][name] = {"error": repr(e)}
            print(f"[bench] secondary {name}: {out['secondary'][name]}", file=sys.stderr, flush=True)
    if not args.no_cpu_baseline:
        print("[bench] timing the CPU oracle on a bounded sample", file=sys.stderr, flush=True)
        out["cpu_baseline"] = cpu_baseline(w, b, args.cpu_budget)
    print(json.dumps(out))
    return 0


if __name__ == "__main__":
    sys.exit(main())
