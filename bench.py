"""Benchmark of the binarized-GCN inference path on one MI355X.

    python bench.py [--gpus 1] [--steps K] [--warmup W] [--workload 5]

A step is one whole forward pass (every layer: sign pack, binary GEMM, CSR
aggregation) over a seeded synthetic workload whose inputs, packed weights
and workspace are already resident in device memory.  The pass is timed
twice, as eager calls and as a HIP-graph replay (checked bit-equal to the
eager pass first); the faster loop gives the reported value (--mode).  A
third timing ("cold_ms_per_step") runs each pass after a 512 MiB write that
evicts the last-level cache and the L2s, so the inputs come from HBM; it is
reported beside the value, not as it.  The default workload is the largest
one: the products-shaped graph (2,449,029 nodes, 126,149,029 CSR entries of
A + I, 100 -> 256 -> 256 -> 47, mean aggregation); the other five (the
sixth a two-weight GraphSAGE model) are selectable with --workload.

Prints one JSON line.  Besides the forward-pass throughput it carries
 - "kernels":  each layer's steps timed alone through their entry points
   (HIP events around a graph replay of --kernel-reps back-to-back calls on
   the launch stream); an aggregation step is all of its kernels (one for
   layers of at most 64 columns, aggregation and fix-up for wider 8-bit
   layers, plus a row plan on the exact-product path).  A layer whose
   aggregation gathers packed signs in the pass ("spmm_sign") has no entry
   point of its own: its time is that of a forward pass over the layer (and
   the next, where only a fused layer gathers signs) less its other steps.
   "in_pass" is whether the forward pass launches the step: a fused layer
   leaves the next one's signs or products, so its pack, or pack and GEMM, are
   not launched;
 - "roofline": the dominant kernel (largest share of a forward pass, among
   those it launches) against its bound: HBM bytes for pack / aggregation
   (each array counted once; the aggregation entries also carry the gather
   model, every edge reading its source's whole row), sign products per second
   for the binary GEMM and the aggregation of signs, against the vector ALUs'
   bit operations or the matrix cores' 4-bit products, whichever it runs on;
   "traffic" is the counter-measured HBM bytes of that call
   (profiles/hbm_traffic_<workload>.md) while the kernel sources match, and
   "traffic_gbs" / "traffic_frac" those bytes over the call's average time
   (against 8 TB/s);
   "cold" is the same entry point timed after cache-evicting writes;
 - "bgemm_ab": the binary GEMM of every layer shape run with both
   algorithms (XOR + bit count on the vector ALUs, +-1 int8 on the matrix
   cores) on the same random sign bits, checked equal, each against its
   own peak in sign products per second;
 - "paper_theoretical": the paper's analytic cycle-operation and size
   ratios for this workload (theory, quoted as such), beside the ratio of
   the fp32 features to the packed sign words this library stores;
 - "cpu_baseline": the plain CPU oracle timed on this host: whole forward
   passes of the same workload, repeated for --cpu-budget seconds (a
   single pass when one takes longer), with the thread count and the host
   CPU model; for graphs of at most 200 K nodes also on one thread
   ("single_thread").

    python bench.py --bgemm-ab

runs only the two-algorithm comparison, over the layer shapes of all five
workloads, and prints it as one JSON line;

    python bench.py --backward [--workload N]

times the back propagation of every layer (bigcn_layer_backward) instead.
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

HBM_PEAK_GBS = 8000.0
# 256 CUs x 4 SIMD x 16 lanes x 2.4 GHz = 39.3 T lane-ops/s; the popcount
# GEMM needs 2 XOR + 2 bit-count lane-ops per 64 sign products.
VALU_BITOP_PEAK = 256 * 4 * 16 * 2.4e9 * 16
# Dense int8 MFMA: 5.0 P ops/s = 2.5 P multiply-adds/s, one sign product each.
MFMA_I8_BITOP_PEAK = 2.5e15
# Dense 4-bit floats: twice that (32 x 32 x 64 products in 32 cycles of a SIMD).
MFMA_E2M1_BITOP_PEAK = 5.0e15
METRIC = "nodes/sec full Bi-GCN forward; bGEMM bit-ops/s; SpMM/pack HBM GB/s vs peak"
COPY_BYTES = 256 << 20   # calibration copy of the byte counters


def log(msg):
    print(msg, file=sys.stderr, flush=True)


def words(k):
    return (k + 63) // 64


def kernel_specs(w, ldF, ldc):
    """Algorithmic work of each kernel of one forward pass, in the units of
    the hot-path scope: every array read or written once, the products as
    16-bit integers in rows of d rounded up to 8 (the library stores most of
    them as 8-bit half-codes, so these are the bytes the method needs, not
    the bytes this implementation moves):
      pack   N*K*4 + N*Kw*8 + N*4 (+ 2*K*4 for mu, rstd on layer 0)
      bGEMM  N*K*d sign products; N*Kw*8 + d*Kw*8 + N*ldc*2 bytes
      SpMM   8(N+1) + 4 nnz + 4N + 2 N ldc + 4 N d bytes (row pointers,
             column indices, scales, products, output); 2 nnz d flops."""
    n, nnz = w.graph.n, w.graph.nnz
    specs = []
    for l, wt in enumerate(w.weights_t):
        d, K = wt.shape
        kw = words(K)
        ldc_l = (d + 7) // 8 * 8
        pack_bytes = n * K * 4 + n * kw * 8 + n * 4 + (2 * K * 4 if l == 0 else 0)
        gemm_ops = n * K * d
        gemm_bytes = n * kw * 8 + d * kw * 8 + n * ldc_l * 2
        spmm_bytes = 8 * (n + 1) + 4 * nnz + 4 * n + 2 * n * ldc_l + 4 * n * d
        specs.append(dict(layer=l, K=K, d=d, pack_bytes=pack_bytes, gemm_ops=gemm_ops,
                          gemm_bytes=gemm_bytes, spmm_bytes=spmm_bytes,
                          spmm_flops=2 * nnz * d))
    return specs


def time_calls(fn, reps, torch):
    """Average GPU duration of one fn() call: `reps` calls are captured into a
    HIP graph and replayed between two HIP events on the launch stream, so no
    host launch gap falls inside the measured interval."""
    fn()                                   # warm up (first-touch, code load)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        for _ in range(reps):
            fn()
    graph.replay()                         # warm replay
    torch.cuda.synchronize()
    start = torch.cuda.Event(enable_timing=True)
    end = torch.cuda.Event(enable_timing=True)
    start.record()
    graph.replay()
    end.record()
    torch.cuda.synchronize()
    return start.elapsed_time(end) / reps * 1e-3


FLUSH_BYTES = 512 << 20   # twice the 256 MB last-level cache
COLD_REPS = 20


def time_cold(fn, reps, torch, flush):
    """Average GPU duration of one fn() call with cold caches: before each
    call a 512 MiB write (a fill kernel, outside the timed interval) evicts
    the last-level cache and every L2, so fn's inputs come from HBM."""
    fn()
    torch.cuda.synchronize()
    total = 0.0
    for i in range(reps):
        flush.fill_(i & 0xFF)
        start = torch.cuda.Event(enable_timing=True)
        end = torch.cuda.Event(enable_timing=True)
        start.record()
        fn()
        end.record()
        torch.cuda.synchronize()
        total += start.elapsed_time(end)
    return total / reps * 1e-3


def gemm_peak(q8, n, d, K, bg):
    """Peak sign products per second of the unit a binary GEMM step runs on."""
    if q8:
        return MFMA_E2M1_BITOP_PEAK if bg._lib.gemm_on_matrix_cores(n, d, K) else VALU_BITOP_PEAK
    return MFMA_I8_BITOP_PEAK if n >= 65536 and K >= 256 and d <= 256 else VALU_BITOP_PEAK


def bgemm_ab(shapes, reps, torch, bg, dev):
    """Both binary-GEMM algorithms on each (M, N, K): seeded random sign bits
    (pad bits zero), results compared bit for bit, durations from time_calls."""
    out = []
    for M, N, K in shapes:
        kw = words(K)
        gen = torch.Generator(device=dev)
        gen.manual_seed(M * 7919 + N * 31 + K)
        F = torch.randint(-2 ** 62, 2 ** 62, (M, kw), dtype=torch.int64, device=dev,
                          generator=gen)
        B = torch.randint(-2 ** 62, 2 ** 62, (N, kw), dtype=torch.int64, device=dev,
                          generator=gen)
        if K % 64:
            F[:, -1] &= (1 << (K % 64)) - 1
            B[:, -1] &= (1 << (K % 64)) - 1
        dt = torch.float16 if K <= 2048 else torch.int16
        res, rec = {}, dict(M=M, N=N, K=K, sign_products=M * N * K)
        for algo, peak in (("popcount", VALU_BITOP_PEAK), ("mfma_i8", MFMA_I8_BITOP_PEAK)):
            C = torch.empty((M, N), dtype=dt, device=dev)
            t = time_calls(lambda: bg.bigcn_bgemm(F, B, K, C, algo=algo), reps, torch)
            res[algo] = C
            rec[algo] = dict(us=round(t * 1e6, 3), tbitops=round(M * N * K / t / 1e12, 2),
                             frac=round(M * N * K / t / peak, 4))
        rec["equal"] = bool(torch.equal(res["popcount"], res["mfma_i8"]))
        rec["faster"] = min(("popcount", "mfma_i8"), key=lambda a: rec[a]["us"])
        out.append(rec)
        log("  bgemm %8d x %3d x %4d: popcount %9.2f us  mfma_i8 %9.2f us  equal=%s" % (
            M, N, K, rec["popcount"]["us"], rec["mfma_i8"]["us"], rec["equal"]))
        del F, B, res
    return out


def measured_traffic(workload_name, layer, entry):
    """HBM bytes (read + written) of one entry-point call, from the committed
    counter summary profiles/hbm_traffic_<workload>.md, or None when there is
    none or the kernel / launch sources changed since it was taken (every device
    source of the forward pass that is there)."""
    import hashlib
    import re
    path = os.path.join(ROOT, "profiles", "hbm_traffic_%s.md" % workload_name)
    if not os.path.exists(path):
        return None
    m = re.search(r"```json\n(.*?)\n```", open(path).read(), re.S)
    if m is None:
        return None
    rec = json.loads(m.group(1))
    h = hashlib.sha256()
    for src in ("bigcn_kernels.hip", "bigcn_api.hip", "bigcn_e2m1.hip", "bigcn_device.h",
                "bigcn_internal.h"):
        src = os.path.join(ROOT, "paper_2010_07565_amd", "csrc", src)
        if os.path.exists(src):
            with open(src, "rb") as f:
                h.update(f.read())
    if rec.get("sources_sha256") != h.hexdigest():
        return None
    for e in rec["entries"]:
        if e["layer"] == layer and e["entry"] == entry:
            return e["fetch_bytes"] + e["write_bytes"]
    return None


def backward_bench(w, model, x, rowptr, colidx, args, torch, bg, dev):
    """Every layer's bigcn_layer_backward on the workload's shapes: layer 0
    reads the features, deeper layers a seeded N(0,1) stand-in input, the
    incoming gradient is seeded N(0, 0.05^2).  All outputs are requested
    (dH, dH~, dW, dW~, db, dzeta), in the model's source order when it has
    one.  Per-layer durations from time_calls; a step is the whole backward
    pass (the sum)."""
    import numpy as np
    import workloads
    g = w.graph
    if w.weights_self_t is not None:
        raise SystemExit("bench.py --backward: the back propagation covers the "
                         "graph-convolution layer (workloads 1-5)")
    layers = []
    total = 0.0
    for l, wt in enumerate(w.weights_t):
        d_out, d_in = wt.shape
        h = x if l == 0 else torch.from_numpy(
            workloads.layer_input(g.n, d_in, seed=3000 + l)).to(dev)
        G = torch.from_numpy((np.random.default_rng(50 + l).standard_normal(
            (g.n, d_out)) * 0.05).astype(np.float32)).to(dev)
        wt_t = torch.from_numpy(wt).to(dev)
        ly = model.layers[l]
        outs = dict(dh=torch.empty((g.n, d_in), device=dev),
                    dh_tilde=torch.empty((g.n, d_in), device=dev),
                    dwt_tilde=torch.empty((d_out, d_in), device=dev),
                    db=torch.empty(d_out, device=dev),
                    dzeta=torch.empty((g.n, d_out), device=dev))
        dwt = torch.empty((d_out, d_in), device=dev)
        ws = torch.empty(bg.layer_backward_workspace_bytes(g.n, g.nnz, d_in, d_out),
                         dtype=torch.uint8, device=dev)
        t = time_calls(lambda: bg.bigcn_layer_backward(rowptr, colidx, h, wt_t, ly.wbits,
                                                       ly.alpha, G, dwt, ws, w.norm,
                                                       slot=model.slot,
                                                       colslot=model.colslot, **outs),
                       args.kernel_reps, torch)
        total += t
        flops = 2.0 * 2.0 * g.n * d_in * d_out          # dW~ and dH~ products
        layers.append(dict(layer=l, d_in=d_in, d_out=d_out, us=round(t * 1e6, 3),
                           gflops=round(flops / t / 1e9, 1)))
        log("  backward L%d %d->%d: %.2f us (%.0f GFLOP/s for dW~ and dH~)" % (
            l, d_in, d_out, t * 1e6, flops / t / 1e9))
    return {"metric": "nodes/sec full Bi-GCN backward (Alg. 1, Eqs. (14)-(15))",
            "value": round(g.n / total, 1), "unit": "nodes/s",
            "ms_per_step": round(total * 1e3, 5), "workload": w.name, "layers": layers,
            "data": "synthetic (seeded inputs and incoming gradients)"}


def source_order(model, torch):
    """The forward pass's source order: (inverse permutation, column slots),
    or (None, column indices) for a model without one.  The per-entry-point
    calls run the aggregation on products and scales moved into that order
    (a copy outside every timed interval): the layout the forward pass
    gathers from."""
    if model.slot is None:
        return None, model.colidx
    order = torch.empty(model.n, dtype=torch.int64, device=model.slot.device)
    order[model.slot.long()] = torch.arange(model.n, device=model.slot.device)
    return order, model.colslot


def to_source_order(order, *ts):
    """Rows of each tensor moved to their slots (nothing without an order)."""
    if order is not None:
        for t in ts:
            t.copy_(t[order])


def sign_pass(w, model, l, h, m0, r0, rowptr, colidx, torch, bg, dev):
    """A forward pass over layer l, which gathers packed signs, and over the next
    too where only a fused layer does: (call, layer l's output, layers in it)."""
    g = w.graph
    d = model.layers[l].d_out
    span = 1 if bg._lib.forward_route(g.n, g.nnz, model.layers[l:l + 1])[0]["signs"] else 2
    out = torch.empty((g.n, d), dtype=torch.float32, device=dev)

    def call_of(layers, res):
        ws = torch.empty(bg.forward_workspace_bytes(g.n, g.nnz, layers), dtype=torch.uint8,
                         device=dev)
        return lambda: bg.bigcn_forward(rowptr, colidx, h, layers, res, ws, m0, r0, w.norm,
                                        slot=model.slot, colslot=model.colslot)
    one = call_of([model.layers[l]], out)
    if span == 1:
        return one, out, 1
    one()                                  # (the output, by the code aggregation)
    res = torch.empty((g.n, model.layers[l + 1].d_out), dtype=torch.float32, device=dev)
    return call_of(model.layers[l:l + 2], res), out, 2


def traffic_probe(w, model, x, rowptr, colidx, torch, bg, dev):
    """One eager call of every per-layer entry point, in the order the
    kernel table times them (for a layer that gathers signs the pack and the
    forward pass of sign_pass), then one 256 MiB device copy of known size."""
    g = w.graph
    route = bg._lib.forward_route(g.n, g.nnz, model.layers)
    kwmax = max(words(wt.shape[1]) for wt in w.weights_t)
    ldF = (kwmax + 1) // 2 * 2
    F = torch.empty((g.n, ldF), dtype=torch.int64, device=dev)
    gs = torch.empty(g.n, dtype=torch.float32, device=dev)
    ldc = max(256, (max(wt.shape[0] for wt in w.weights_t) + 7) // 8 * 8)
    C = torch.empty((g.n, ldc), dtype=torch.float16, device=dev)
    C8 = torch.empty((g.n, 256), dtype=torch.int8, device=dev)
    ws = torch.empty(max(bg.spmm_workspace_bytes(g.n, g.nnz, wt.shape[0])
                         for wt in w.weights_t), dtype=torch.uint8, device=dev)
    mu_t = torch.from_numpy(w.mu).to(dev)
    rstd_t = torch.from_numpy(w.rstd).to(dev)
    order, src = source_order(model, torch)
    h = x
    for l, ly in enumerate(model.layers):
        K, d = ly.d_in, ly.d_out
        kw = words(K)
        out = torch.empty((g.n, d), dtype=torch.float32, device=dev)
        torch.cuda.synchronize()
        log("probe layer %d: pack" % l)
        bg.bigcn_binarize_pack(h, F[:, :kw], gs, mu_t if l == 0 else None,
                               rstd_t if l == 0 else None, rowptr, w.norm)
        if route[l]["signs"]:
            log("probe layer %d: spmm_sign" % l)
            call, out, _ = sign_pass(w, model, l, h, mu_t if l == 0 else None,
                                     rstd_t if l == 0 else None, rowptr, colidx, torch, bg, dev)
            call()
        elif bg.q8_supported(g.n, d, K):
            W = bg.q8_row(d)
            c8 = C8.view(-1)[:g.n * W].view(g.n, W)
            c16 = C.view(-1)[:g.n * W].view(g.n, W)
            log("probe layer %d: bgemm_q8, spmm_q8" % l)
            bg.bigcn_bgemm_q8(F[:, :kw], ly.wbits, K, c8, c16, gs)
            if ly.wbits_self is not None:
                Cs = torch.empty((g.n, (d + 7) // 8 * 8), dtype=torch.float16, device=dev)
                bg.bigcn_bgemm(F[:, :kw], ly.wbits_self, K, Cs[:, :d])
                torch.cuda.synchronize()
                to_source_order(order, c8, c16, gs, Cs)
                torch.cuda.synchronize()
                bg.bigcn_spmm_csr_sage_q8(rowptr, src, gs, c8, c16, K, ly.alpha, Cs,
                                          ly.alpha_self, out, ws, ly.bias, ly.act, d=d)
            else:
                torch.cuda.synchronize()
                to_source_order(order, c8, c16, gs)
                torch.cuda.synchronize()
                bg.bigcn_spmm_csr_q8(rowptr, src, gs, c8, c16, K, ly.alpha, out, ws,
                                     ly.bias, w.norm, ly.act, d=d)
        else:
            log("probe layer %d: bgemm, spmm" % l)
            bg.bigcn_bgemm(F[:, :kw], ly.wbits, K, C[:, :d])
            torch.cuda.synchronize()
            to_source_order(order, C, gs)
            torch.cuda.synchronize()
            bg.bigcn_spmm_csr(rowptr, src, gs, C, ly.alpha, out, ws, ly.bias, w.norm,
                              ly.act, d=d)
        h = out
    torch.cuda.synchronize()
    src = torch.ones(COPY_BYTES // 4, dtype=torch.float32, device=dev)
    dst = torch.empty_like(src)
    torch.cuda.synchronize()
    log("probe: copy of %d bytes" % COPY_BYTES)
    dst.copy_(src)
    torch.cuda.synchronize()
    print(json.dumps({"traffic_probe": w.name, "copy_bytes": COPY_BYTES}), flush=True)


def host_cpu_model():
    """The host CPU's model name (first 'model name' of /proc/cpuinfo)."""
    try:
        with open("/proc/cpuinfo") as f:
            for line in f:
                if line.startswith("model name"):
                    return line.split(":", 1)[1].strip()
    except OSError:
        pass
    return None


def _time_oracle_passes(w, budget_s):
    """Whole oracle forward passes of workload w, repeated until budget_s has
    elapsed (one pass when a single pass takes longer).  Each layer's
    double-precision arrays are dropped as soon as the next layer has its
    input, as a caller of the per-layer chain may.  Returns (passes, s)."""
    import oracle

    g = w.graph
    sage = w.weights_self_t is not None
    t0 = time.time()
    reps = 0
    while True:
        if sage:
            chain = oracle.sage_forward_layers(g.rowptr, g.colidx, w.x, w.weights_self_t,
                                               w.weights_t, w.biases, mu=w.mu, rstd=w.rstd)
        else:
            chain = oracle.forward_layers(g.rowptr, g.colidx, w.norm, w.x, w.weights_t,
                                          w.biases, mu=w.mu, rstd=w.rstd)
        for _ in chain:
            pass
        reps += 1
        if time.time() - t0 >= budget_s or reps >= 10_000:
            break
    return reps, time.time() - t0


def cpu_baseline(w, budget_s=10.0, single_thread_max_nodes=200_000):
    """The oracle on this host, whole forward passes of the same workload on
    every OpenMP thread (nodes per second over the timed passes).  Graphs of
    at most single_thread_max_nodes nodes are also timed on one thread."""
    import oracle

    g = w.graph
    cores = oracle.threads()
    reps, dt = _time_oracle_passes(w, budget_s)
    out = dict(value=g.n * reps / dt, unit="nodes/s", cores=cores, kind="oracle",
               cpu_model=host_cpu_model(),
               sample="whole %d-node forward pass x %d in %.1f s (plain oracle, not a "
                      "tuned CPU library; %d OpenMP threads)" % (g.n, reps, dt, cores))
    if g.n <= single_thread_max_nodes:
        oracle.set_threads(1)
        try:
            reps1, dt1 = _time_oracle_passes(w, budget_s)
        finally:
            oracle.set_threads(cores)
        out["single_thread"] = dict(
            value=g.n * reps1 / dt1, unit="nodes/s", cores=1,
            sample="whole %d-node forward pass x %d in %.1f s on one thread" % (g.n, reps1, dt1))
    return out


def main():
    ap = argparse.ArgumentParser(description=__doc__.split("\n")[0])
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=200)
    ap.add_argument("--warmup", type=int, default=20)
    ap.add_argument("--workload", type=int, default=5, choices=[1, 2, 3, 4, 5, 6])
    ap.add_argument("--kernel-reps", type=int, default=20)
    ap.add_argument("--cpu-budget", type=float, default=10.0)
    ap.add_argument("--no-cpu-baseline", action="store_true")
    ap.add_argument("--mode", choices=["best", "graph", "eager"], default="best",
                    help="which timed loop gives the reported value: the faster of "
                         "the two (default), the HIP-graph replay, or eager calls")
    ap.add_argument("--forward-only", action="store_true",
                    help="time the forward pass only (no per-kernel table, no "
                         "algorithm comparison, no CPU baseline): for profiling")
    ap.add_argument("--traffic-probe", action="store_true",
                    help="call each entry point of the workload once, eagerly, then "
                         "copy 256 MiB device to device (the counter calibration "
                         "kernel): the program profiled for HBM byte counters")
    ap.add_argument("--backward", action="store_true",
                    help="time the back propagation of every layer of the workload "
                         "(Alg. 1, Eqs. (14)-(15)) instead of the forward pass")
    ap.add_argument("--bgemm-ab", action="store_true",
                    help="only compare the two binary-GEMM algorithms on every "
                         "workload's layer shapes")
    args = ap.parse_args()

    if args.gpus != 1:
        print("bench.py: the path runs on a single GPU; --gpus %d is not supported "
              "(the multi-GPU design is described, not built)" % args.gpus,
              file=sys.stderr)
        sys.exit(2)

    import numpy as np
    import torch
    import workloads
    import paper_2010_07565_amd as bg

    assert torch.cuda.is_available(), "bench.py needs a GPU"
    dev = torch.device("cuda:0")
    if args.bgemm_ab:
        shapes = []
        for c in workloads.CONFIGS.values():
            for K, d in zip(c["dims"][:-1], c["dims"][1:]):
                shapes.append((c["n"], d, K))
        ab = bgemm_ab(shapes, args.kernel_reps, torch, bg, dev)
        assert all(r["equal"] for r in ab), "binary-GEMM algorithms disagree"
        print(json.dumps({"bgemm_ab": ab, "peaks_tbitops": {
            "popcount": VALU_BITOP_PEAK / 1e12, "mfma_i8": MFMA_I8_BITOP_PEAK / 1e12}}),
              flush=True)
        return
    t0 = time.time()
    w = workloads.make_workload(args.workload)
    g = w.graph
    log("workload %d (%s) generated in %.1f s: %s" % (args.workload, w.name, time.time() - t0,
                                                        workloads.degree_summary(g)))

    rowptr = torch.from_numpy(g.rowptr).to(dev)
    colidx = torch.from_numpy(g.colidx).to(dev)
    x = torch.from_numpy(w.x).to(dev)
    model = bg.BiGCN(rowptr, colidx, w.weights_t, w.biases, norm=w.norm, mu=w.mu,
                     rstd=w.rstd, device=dev, weights_self_t=w.weights_self_t)
    torch.cuda.synchronize()
    if args.traffic_probe:
        traffic_probe(w, model, x, rowptr, colidx, torch, bg, dev)
        return
    if args.backward:
        print(json.dumps(backward_bench(w, model, x, rowptr, colidx, args, torch, bg, dev)),
              flush=True)
        return

    # ---- the timed forward passes: eager calls, then the same pass replayed
    # from a HIP graph (the serving loop); the graph's output is checked
    # against the eager one bit for bit before it is timed.
    def timed(fn, steps, warmup):
        for _ in range(warmup):
            fn()
        torch.cuda.synchronize()
        t = time.perf_counter()
        for _ in range(steps):
            fn()
        torch.cuda.synchronize()
        return (time.perf_counter() - t) / steps

    eager_s = timed(lambda: model.forward(x), args.steps, args.warmup)
    eager_out = model.out.clone()
    replay = model.capture(x)
    replay()
    torch.cuda.synchronize()
    assert torch.equal(model.out, eager_out), "graph replay differs from the eager pass"
    graph_s = timed(replay, args.steps, args.warmup)
    flush = torch.empty(FLUSH_BYTES, dtype=torch.uint8, device=dev)
    cold_s = time_cold(lambda: model.forward(x), COLD_REPS, torch, flush)
    if args.mode == "best":
        mode = "hip_graph_replay" if graph_s <= eager_s else "eager"
    else:
        mode = "hip_graph_replay" if args.mode == "graph" else "eager"
    step_s = graph_s if mode == "hip_graph_replay" else eager_s
    ms = step_s * 1e3
    nodes_per_s = g.n / step_s
    log("forward: eager %.4f ms/step, graph replay %.4f ms/step -> %.4g nodes/s" % (
        eager_s * 1e3, graph_s * 1e3, nodes_per_s))

    if args.forward_only:
        print(json.dumps({"metric": METRIC, "value": round(nodes_per_s, 1), "unit": "nodes/s",
                          "ms_per_step": round(ms, 5), "workload": w.name,
                          "mode": mode, "eager_ms_per_step": round(eager_s * 1e3, 5),
                          "graph_ms_per_step": round(graph_s * 1e3, 5)}), flush=True)
        return

    # ---- each kernel alone, through its entry point, same shapes and ld's
    L = len(w.weights_t)
    kwmax = max(words(wt.shape[1]) for wt in w.weights_t)
    ldF = (kwmax + 1) // 2 * 2
    ldc = (max(wt.shape[0] for wt in w.weights_t) + 7) // 8 * 8
    F = torch.empty((g.n, ldF), dtype=torch.int64, device=dev)
    gs = torch.empty(g.n, dtype=torch.float32, device=dev)
    C = torch.empty((g.n, max(256, ldc)), dtype=torch.float16, device=dev)
    C8 = torch.empty((g.n, 256), dtype=torch.int8, device=dev)
    ws = torch.empty(max(bg.spmm_workspace_bytes(g.n, g.nnz, wt.shape[0])
                         for wt in w.weights_t), dtype=torch.uint8, device=dev)
    mu_t = torch.from_numpy(w.mu).to(dev)
    rstd_t = torch.from_numpy(w.rstd).to(dev)
    specs = kernel_specs(w, ldF, ldc)
    kernels = []
    calls = {}
    order, src = source_order(model, torch)
    route = bg._lib.forward_route(g.n, g.nnz, model.layers)
    h = x
    reps = args.kernel_reps
    for l, ly in enumerate(model.layers):
        K, d = ly.d_in, ly.d_out
        out = torch.empty((g.n, d), dtype=torch.float32, device=dev)
        kw = words(K)
        m0 = mu_t if l == 0 else None
        r0 = rstd_t if l == 0 else None
        f_pack = (lambda h=h, kw=kw, m0=m0, r0=r0: bg.bigcn_binarize_pack(
            h, F[:, :kw], gs, m0, r0, rowptr, w.norm))
        t_pack = time_calls(f_pack, reps, torch)
        q8 = bg.q8_supported(g.n, d, K)
        sage = ly.wbits_self is not None
        t_self = None
        # what the pass launches of this layer: not what the layer before leaves
        left = route[l - 1]["leaves"] if l > 0 else None
        if route[l]["signs"]:
            f_layer, out, span = sign_pass(w, model, l, h, m0, r0, rowptr, colidx, torch, bg, dev)
            row = bg._lib.sign_row_bytes(K)
            work = 8 * (g.n + 1) + 4 * g.nnz + 4 * g.n + g.n * row + 4 * g.n * d
            gather = g.nnz * (8 + row) + g.n * d * 4
            kernels += [
                dict(kernel="pack", layer=l, us=t_pack * 1e6, bound="hbm",
                     achieved=specs[l]["pack_bytes"] / t_pack / 1e9, unit="GB/s",
                     peak=HBM_PEAK_GBS, work=specs[l]["pack_bytes"], in_pass=left is None),
                dict(kernel="spmm_sign", layer=l, us=time_calls(f_layer, reps, torch) * 1e6,
                     bound="alu", unit="Tbitop/s", peak=MFMA_E2M1_BITOP_PEAK / 1e12,
                     ops=g.nnz * K * d, work=g.nnz * K * d, bytes=work, gather_bytes=gather,
                     in_pass=True, span=span)]
            calls[(l, "pack")], calls[(l, "spmm")] = f_pack, f_layer
            h = out
            continue
        if q8:
            # the forward keeps these products as 8-bit half-codes, in rows
            # of q8_row(d) entries
            W = bg.q8_row(d)
            c8 = C8.view(-1)[:g.n * W].view(g.n, W)
            c16 = C.view(-1)[:g.n * W].view(g.n, W)
            f_gemm = (lambda kw=kw, ly=ly, K=K, c8=c8, c16=c16: bg.bigcn_bgemm_q8(
                F[:, :kw], ly.wbits, K, c8, c16, gs))
            t_gemm = time_calls(f_gemm, reps, torch)
            if sage:   # the self products, exact in half, and the GraphSAGE aggregation
                Cs = torch.empty((g.n, (d + 7) // 8 * 8), dtype=torch.float16, device=dev)
                f_self = (lambda kw=kw, ly=ly, K=K, Cs=Cs, d=d: bg.bigcn_bgemm(
                    F[:, :kw], ly.wbits_self, K, Cs[:, :d]))
                t_self = time_calls(f_self, reps, torch)

                def prep(f_pack=f_pack, f_gemm=f_gemm, f_self=f_self, c8=c8, c16=c16, Cs=Cs):
                    f_pack()
                    f_gemm()
                    f_self()
                    torch.cuda.synchronize()
                    to_source_order(order, c8, c16, gs, Cs)
                prep()
                f_spmm = (lambda c8=c8, c16=c16, K=K, ly=ly, Cs=Cs, out=out, d=d:
                          bg.bigcn_spmm_csr_sage_q8(rowptr, src, gs, c8, c16, K, ly.alpha, Cs,
                                                    ly.alpha_self, out, ws, ly.bias, ly.act,
                                                    d=d))
                t_spmm = time_calls(f_spmm, reps, torch)
            else:
                def prep(f_pack=f_pack, f_gemm=f_gemm, c8=c8, c16=c16):
                    f_pack()
                    f_gemm()
                    torch.cuda.synchronize()
                    to_source_order(order, c8, c16, gs)
                prep()
                f_spmm = (lambda c8=c8, c16=c16, K=K, ly=ly, out=out, d=d:
                          bg.bigcn_spmm_csr_q8(rowptr, src, gs, c8, c16, K, ly.alpha, out,
                                               ws, ly.bias, w.norm, ly.act, d=d))
                t_spmm = time_calls(f_spmm, reps, torch)
        else:
            f_gemm = (lambda kw=kw, ly=ly, K=K, d=d: bg.bigcn_bgemm(F[:, :kw], ly.wbits, K,
                                                                     C[:, :d]))
            t_gemm = time_calls(f_gemm, reps, torch)

            def prep(f_pack=f_pack, f_gemm=f_gemm):
                f_pack()
                f_gemm()
                torch.cuda.synchronize()
                to_source_order(order, C, gs)
            prep()
            f_spmm = (lambda ly=ly, out=out, d=d: bg.bigcn_spmm_csr(
                rowptr, src, gs, C, ly.alpha, out, ws, ly.bias, w.norm, ly.act, d=d))
            t_spmm = time_calls(f_spmm, reps, torch)
        s = specs[l]
        calls[(l, "pack")], calls[(l, "gemm")], calls[(l, "spmm")] = f_pack, f_gemm, f_spmm
        calls[(l, "prep")] = prep
        kernels += [
            dict(kernel="pack", layer=l, us=t_pack * 1e6, bound="hbm",
                 achieved=s["pack_bytes"] / t_pack / 1e9, unit="GB/s", peak=HBM_PEAK_GBS,
                 work=s["pack_bytes"], in_pass=left is None),
            dict(kernel="bgemm_q8" if q8 else "bgemm", layer=l, us=t_gemm * 1e6, bound="alu",
                 achieved=s["gemm_ops"] / t_gemm / 1e12, unit="Tbitop/s",
                 peak=gemm_peak(q8, g.n, d, K, bg) / 1e12, work=s["gemm_ops"],
                 bytes=s["gemm_bytes"], hbm_gbs=s["gemm_bytes"] / t_gemm / 1e9,
                 in_pass=left != "products"),
            dict(kernel=("spmm_sage_q8" if sage else "spmm_q8") if q8 else "spmm", layer=l,
                 us=t_spmm * 1e6, bound="hbm",
                 achieved=(s["spmm_bytes"] + (g.n * d * 2 if sage else 0)) / t_spmm / 1e9,
                 unit="GB/s", peak=HBM_PEAK_GBS,
                 work=s["spmm_bytes"] + (g.n * d * 2 if sage else 0),
                 # every edge re-reads its source's product row (whole row of
                 # the stored layout), column index and scale
                 gather_bytes=g.nnz * (8 + (bg.q8_row(d) if q8 else 2 * ((d + 7) // 8 * 8)))
                 + g.n * d * 4,
                 gather_gbs=(g.nnz * (8 + (bg.q8_row(d) if q8 else 2 * ((d + 7) // 8 * 8)))
                             + g.n * d * 4) / t_spmm / 1e9, in_pass=True),
        ]
        if t_self is not None:
            kernels.append(dict(kernel="bgemm_self", layer=l, us=t_self * 1e6, bound="alu",
                                achieved=s["gemm_ops"] / t_self / 1e12, unit="Tbitop/s",
                                peak=VALU_BITOP_PEAK / 1e12, work=s["gemm_ops"],
                                bytes=g.n * kw * 8 + d * kw * 8 + g.n * d * 2,
                                hbm_gbs=(g.n * kw * 8 + g.n * d * 2) / t_self / 1e9,
                                in_pass=d <= 64))   # (wider: formed in the epilogue)
        h = out
    us = {(k["layer"], k["kernel"].split("_")[0]): k["us"] for k in kernels
          if k["kernel"] != "bgemm_self"}
    for k in kernels:
        if k["kernel"] == "spmm_sign":     # the layer's pass less its other steps
            l = k["layer"]
            k["us"] -= us[(l, "pack")]
            if k.pop("span") == 2:
                k["us"] -= us.get((l + 1, "bgemm"), 0.0) + us[(l + 1, "spmm")]
            k["achieved"] = k.pop("ops") / k["us"] * 1e6 / 1e12
            k["gather_gbs"] = k["gather_bytes"] / k["us"] * 1e6 / 1e9
    for k in kernels:
        k["frac"] = k["achieved"] / k["peak"]
        log("  L%d %-5s %9.2f us  %8.1f %s  (%.1f%% of peak)" % (
            k["layer"], k["kernel"], k["us"], k["achieved"], k["unit"], 100 * k["frac"]))
    dom = max((k for k in kernels if k["in_pass"]), key=lambda k: k["us"])
    entry = dom["kernel"].split("_")[0]                  # pack / bgemm / spmm
    traffic = measured_traffic(w.name, dom["layer"], entry)
    # the same entry point with cold caches (inputs from HBM, not from the
    # last-level cache that holds a small graph's whole working set)
    if (dom["layer"], "prep") in calls:   # that layer's own products, in source order
        calls[(dom["layer"], "prep")]()
    cold_us = time_cold(calls[(dom["layer"], "gemm" if entry == "bgemm" else entry)],
                        COLD_REPS, torch, flush) * 1e6
    if dom["kernel"] == "spmm_sign":      # (a pass: its other steps come warm after the pack)
        cold_us -= us[(dom["layer"], "spmm")] - dom["us"]
    cold_achieved = dom["achieved"] * dom["us"] / cold_us
    roofline = dict(kernel="%s (layer %d)" % (dom["kernel"], dom["layer"]), bound=dom["bound"],
                    achieved=round(dom["achieved"], 2), peak=dom["peak"], unit=dom["unit"],
                    frac=round(dom["frac"], 4), traffic=traffic,
                    traffic_unit="bytes per call (HBM read + written)",
                    # the counted bytes over the same average duration: the
                    # rate the memory system actually delivered for this call
                    traffic_gbs=(round(traffic / (dom["us"] * 1e-6) / 1e9, 1)
                                 if traffic is not None else None),
                    traffic_frac=(round(traffic / (dom["us"] * 1e-6) / 1e9 / HBM_PEAK_GBS, 4)
                                  if traffic is not None else None),
                    algorithmic_bytes=dom["work"] if dom["bound"] == "hbm" else dom.get("bytes"),
                    avg_us=round(dom["us"], 3),
                    timing="warm: back-to-back calls (a HIP graph between two HIP events on "
                           "the launch stream)",
                    cold={"avg_us": round(cold_us, 3), "achieved": round(cold_achieved, 2),
                          "frac": round(cold_achieved / dom["peak"], 4),
                          "timing": "each call after a 512 MiB write that evicts the "
                                    "last-level cache and the L2s"})

    ab = bgemm_ab([(g.n, ly.d_out, ly.d_in) for ly in model.layers], reps, torch, bg, dev)
    assert all(r["equal"] for r in ab), "binary-GEMM algorithms disagree"

    cpu = None
    if not args.no_cpu_baseline:
        t = time.time()
        cpu = cpu_baseline(w, args.cpu_budget)
        log("cpu baseline: %s (%.1f s)" % (cpu, time.time() - t))

    dims = [w.weights_t[0].shape[1]] + [wt.shape[0] for wt in w.weights_t]
    from paper_2010_07565_amd import costmodel
    undirected = (g.nnz - g.n) // 2
    wpl = 2 if w.weights_self_t is not None else 1
    if w.weights_self_t is not None:
        undirected = g.nnz // 2                          # A has no self-loops
    theory = costmodel.theoretical_ratios(g.n, undirected, dims, wpl)
    paper = {
        "kind": "the paper's analytic counts (Sec. 5: cycle operations, model and "
                "feature sizes, full precision over binarized) for this workload; "
                "not measurements",
        "cycle_op_speedup": round(theory["cycle_ops"], 2),
        "model_size_ratio": round(theory["model_size"], 2),
        "data_size_ratio": round(theory["data_size"], 2),
        "co_shares": {k: round(v, 3) for k, v in
                      costmodel.co_breakdown(g.n, undirected, dims).items()},
        "quoted": "about 47x fewer cycle operations and about 30x less memory on "
                  "the citation graphs (Sec. 6.3)",
        "stored_feature_ratio": round((g.n * dims[0] * 4) / (g.n * ldF * 8 + g.n * 4), 2),
    }
    rec = {
        "metric": METRIC,
        "value": round(nodes_per_s, 1),
        "unit": "nodes/s",
        "n_gpus": 1,
        "steps": args.steps,
        "warmup": args.warmup,
        "ms_per_step": round(ms, 5),
        "mode": mode,
        "graph_ms_per_step": round(graph_s * 1e3, 5),
        "eager_ms_per_step": round(eager_s * 1e3, 5),
        "cold_ms_per_step": round(cold_s * 1e3, 5),
        "higher_is_better": True,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": "u64 sign bits + fp32",
        "data": "synthetic (seeded %s stand-in)" % w.name,
        "config": {"workload": "%s: %d-layer Bi-GCN %s, %d nodes, %d CSR entries of A+I, "
                               "%s normalisation" % (w.name, L, "-".join(map(str, dims)),
                                                     g.n, g.nnz, w.norm),
                   "nodes": g.n, "nnz": g.nnz, "dims": dims, "norm": w.norm,
                   "parallelism": "single GPU"},
        "kernels": [{k2: (round(v, 4) if isinstance(v, float) else v) for k2, v in k.items()}
                    for k in kernels],
        "roofline": roofline,
        "bgemm_ab": ab,
        "paper_theoretical": paper,
        "cpu_baseline": cpu,
    }
    print(json.dumps(rec), flush=True)


if __name__ == "__main__":
    main()
