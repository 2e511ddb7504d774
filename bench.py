#!/usr/bin/env python3
"""Benchmark of the BitLinear hot path on one MI355X.

    python bench.py [--gpus 1] [--steps K] [--warmup W] [--no-cpu] [--no-decode] [--no-train] [--no-prefill-30b]

Workload at one GPU: the BitNet-6.7B-shaped prefill pair (4096->16384 and 16384->4096 at
M = 2048 tokens, activations N(0,1) with 0.1 % outliers x20, weights N(0, 0.02^2)).
A step is one BitLinear forward (LayerNorm + absmax quantiser + 1-bit x 8-bit MFMA GEMM +
dequantisation, i.e. Eq. 12, 4-5, 7 and 11 of arXiv 2310.11453) through each of the two
layers, inputs and packed weights resident in HBM.  Weight packing (Eq. 1-3) happens once
per weight at inference and is timed separately ("weight_prep").

Prints ONE JSON line.  `value` is prefill TOPS (2*M*N*K summed over the step / step time);
`roofline` describes the dominant kernel (the MFMA GEMM) from HIP-event timing of that
kernel alone inside the timed loop; `decode` reports the packed-weight streaming rate of
the small-M kernel on BitNet-30B-shaped layers; `training` times one forward + straight-through
backward of the 4096->16384 layer at M = 8192; `cpu_baseline` times the CPU oracle on a bounded
sample of the same workload on this machine's host cores.
"""
from __future__ import annotations

import argparse
import ctypes
import json
import sys
import time

import numpy as np

import workloads as wl

HBM_PEAK_GBS = 8000.0
I8_MFMA_PEAK_TOPS = 5000.0

# HBM bytes per launch of the dominant kernel (the 4096->16384 GEMM at M=2048) measured with
# rocprofv3 --pmc FETCH_SIZE / WRITE_SIZE, each scaled by what the same counter reads for a
# plain 256 MiB device copy (x2.000 and x1.000): profiles/gemm_prefill_6p7b_counters.txt.
TRAFFIC_BYTES = {"gemm_prefill_up": int((41129 * 2.000 + 131200 * 1.000) * 1024)}


def gemm_bytes(M, K, N):
    """Algorithmic bytes of GEMM + epilogue: packed weights, int8 codes, fp32 output, gamma."""
    return N * K // 8 + M * K + 4 * M * N + 4 * M


def event_ms(fn, iters, torch):
    start, end = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    start.record()
    for _ in range(iters):
        fn()
    end.record()
    end.synchronize()
    return start.elapsed_time(end) / iters


def graph_ms(fn, launches, replays, torch):
    """Per-call milliseconds of `fn` from `launches` calls captured once into a HIP graph and
    replayed: the kernels run back to back on the device, so kernels of a few microseconds are
    timed at the rate the device runs them, not at the rate Python can enqueue them.  `fn` takes
    the index of the call (callers rotate buffers with it).  Falls back to eager launches."""
    try:
        side = torch.cuda.Stream()
        side.wait_stream(torch.cuda.current_stream())
        with torch.cuda.stream(side):
            for i in range(launches):
                fn(i)
        torch.cuda.current_stream().wait_stream(side)
        torch.cuda.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g):
            for i in range(launches):
                fn(i)
        g.replay()
        torch.cuda.synchronize()
        return event_ms(g.replay, replays, torch) / launches, "HIP graph replay"
    except Exception as exc:  # capture unavailable
        state = {"i": 0}

        def eager():
            fn(state["i"])
            state["i"] += 1

        return event_ms(eager, launches * replays, torch), f"eager ({type(exc).__name__})"


def decode_stacks(bl, torch, dev, decode):
    """The stream / whole-block legs of the decode measurement (added to `decode`)."""
    c3 = wl.CONFIGS[3]
    # Layer stream at the 1.3B shapes: the four projections of 24 layers, four distinct sets of
    # them (604 MB of packed weights, more than L2 + Infinity Cache), enqueued back to back as
    # one HIP graph per batch size; GB/s = algorithmic bytes of all launches / time.
    c2 = wl.CONFIGS[1]
    protos = []
    for li, L2 in enumerate(c2.layers):
        W2 = wl.make_weight(L2.N, L2.K, c2.w_std, wl.seed_for(1, li))
        p2, _, b2 = bl.bitlinear_pack_weights(torch.from_numpy(W2).to(dev))
        protos.append((L2, p2, b2))
        del W2
    n_sets = 4 * 24
    sets = [[(L2, p2.clone(), b2) for (L2, p2, b2) in protos] for _ in range(n_sets)]
    stream = []
    for Md in (1, 4, 16):
        acts = {}
        for K2 in sorted({L2.K for (L2, _, _) in protos}):
            X2 = torch.from_numpy(wl.make_activation(Md, K2, wl.seed_for(1, K2 % 97))).to(dev)
            acts[K2] = bl.bitlinear_quant_act(X2)[:3]
        outs = {L2.name: torch.empty((Md, L2.N), dtype=torch.float32, device=dev)
                for (L2, _, _) in protos}

        def run_stream():
            for layer in sets:
                for (L2, p2, b2) in layer:
                    c_, g_, r_ = acts[L2.K]
                    bl.bitlinear_matmul(c_, g_, r_, p2, L2.N, b2, out=outs[L2.name])

        run_stream()
        torch.cuda.synchronize()
        mode = "eager launches"
        timed = run_stream
        try:
            side = torch.cuda.Stream()
            side.wait_stream(torch.cuda.current_stream())
            with torch.cuda.stream(side):
                run_stream()
            torch.cuda.current_stream().wait_stream(side)
            graph = torch.cuda.CUDAGraph()
            with torch.cuda.graph(graph):
                run_stream()
            ref = {k: v.clone() for k, v in outs.items()}
            graph.replay()
            torch.cuda.synchronize()
            if all(torch.equal(ref[k], outs[k]) for k in outs):
                timed, mode = graph.replay, "one HIP graph of all launches, replayed"
        except Exception as exc:  # capture unavailable: time the eager launches
            mode = f"eager launches (graph capture failed: {type(exc).__name__})"
        timed()
        t = event_ms(timed, 5, torch)
        nbytes = sum(gemm_bytes(Md, L2.K, L2.N) for layer in sets for (L2, _, _) in layer)
        stream.append(dict(M=Md, launches=len(sets) * len(protos), us=t * 1e3,
                           us_per_launch=t * 1e3 / (len(sets) * len(protos)),
                           gbs=nbytes / (t * 1e-3) / 1e9,
                           frac_hbm=nbytes / (t * 1e-3) / 1e9 / HBM_PEAK_GBS, launch=mode))
    decode["layer_stream_1p3b"] = stream

    # One decoding step of the 24-layer stack: LN + quantise + GEMM + dequant through QKV, O,
    # up and down of every layer, each input being the previous output (the attention and the
    # non-linearity between them are left out: only their place in the chain matters here).
    # Four stacks of distinct weights, one HIP graph each, replayed in turn.
    block = []
    for Md in (1, 4, 16):
        h0 = torch.from_numpy(wl.make_activation(Md, 2048, wl.seed_for(1, 50))).to(dev)
        bufs = {L2.name: torch.empty((Md, L2.N), dtype=torch.float32, device=dev)
                for (L2, _, _) in protos}
        wss = {L2.name: torch.empty(bl.workspace_bytes(bl.OP_FORWARD, Md, L2.N, L2.K),
                                    dtype=torch.uint8, device=dev) for (L2, _, _) in protos}

        def run_stack(layers24):
            h = h0
            for layer in layers24:
                for (L2, p2, b2) in layer:
                    x_in = h if h.shape[1] == L2.K else h.view(-1)[:Md * L2.K].view(Md, L2.K)
                    h = bl.bitlinear_forward(x_in, p2, L2.N, b2, out=bufs[L2.name],
                                             workspace=wss[L2.name])
            return h

        stacks = [sets[i * 24:(i + 1) * 24] for i in range(4)]
        ref = run_stack(stacks[0]).clone()
        torch.cuda.synchronize()
        mode, n_launch = "eager launches", None
        runners = [lambda st=st: run_stack(st) for st in stacks]
        try:
            graphs = []
            for st in stacks:
                side = torch.cuda.Stream()
                side.wait_stream(torch.cuda.current_stream())
                with torch.cuda.stream(side):
                    run_stack(st)
                torch.cuda.current_stream().wait_stream(side)
                g2 = torch.cuda.CUDAGraph(keep_graph=True)
                with torch.cuda.graph(g2):
                    run_stack(st)
                graphs.append(g2)
            nodes = ctypes.c_size_t()  # all of them kernels
            if bl.load_library().hipGraphGetNodes(ctypes.c_void_p(graphs[0].raw_cuda_graph()), None,
                                                  ctypes.byref(nodes)) == 0:
                n_launch = nodes.value
            graphs[0].replay()
            torch.cuda.synchronize()
            if torch.equal(ref, bufs["down"]):
                runners, mode = [g2.replay for g2 in graphs], "one HIP graph per stack, replayed"
        except Exception as exc:
            mode = f"eager launches (graph capture failed: {type(exc).__name__})"

        def run_all():
            for r in runners:
                r()

        run_all()
        t = event_ms(run_all, 5, torch) / len(runners)
        nbytes = sum(gemm_bytes(Md, L2.K, L2.N) + 5 * Md * L2.K for (L2, _, _) in protos) * 24
        block.append(dict(M=Md, layers=24, launches=n_launch, us_per_step=t * 1e3,
                          us_per_launch=t * 1e3 / n_launch if n_launch else None,
                          gbs=nbytes / (t * 1e-3) / 1e9, launch=mode))
    decode["block_decode_1p3b"] = block
    del sets, protos

    # The same chain at the 6.7B shapes (d = 4096; the whole 32-layer stack, 0.8 GB of packed
    # weights) and the 30B shapes (d = 7168; eight distinct layers, 0.6 GB), one token: one HIP
    # graph, one launch per projection (the GEMM kernel quantises the row itself).
    for tag, d, n_layers, w_std, sd in (("6p7b", 4096, 32, 0.02, 2), ("30b", 7168, 8, c3.w_std, 3)):
        shapes = [wl.Layer("qkv", d, 3 * d), wl.Layer("o", d, d), wl.Layer("up", d, 4 * d),
                  wl.Layer("down", 4 * d, d)]
        protos3 = []
        for li, L3 in enumerate(shapes):
            W3 = wl.make_weight(L3.N, L3.K, w_std, wl.seed_for(sd, 10 + li))
            p3, _, b3 = bl.bitlinear_pack_weights(torch.from_numpy(W3).to(dev))
            protos3.append((L3, p3, b3))
            del W3
        stack = [[(L3, p3.clone(), b3) for (L3, p3, b3) in protos3] for _ in range(n_layers)]
        h0 = torch.from_numpy(wl.make_activation(1, d, wl.seed_for(sd, 50))).to(dev)
        bufs3 = {L3.name: torch.empty((1, L3.N), dtype=torch.float32, device=dev) for (L3, _, _) in protos3}
        wss3 = {L3.name: torch.empty(bl.workspace_bytes(bl.OP_FORWARD, 1, L3.N, L3.K), dtype=torch.uint8,
                                     device=dev) for (L3, _, _) in protos3}

        def run_stack3():
            h = h0
            for layer in stack:
                for (L3, p3, b3) in layer:
                    x_in = h if h.shape[1] == L3.K else h.view(-1)[:L3.K].view(1, L3.K)
                    h = bl.bitlinear_forward(x_in, p3, L3.N, b3, out=bufs3[L3.name], workspace=wss3[L3.name])
            return h

        ref3 = run_stack3().clone()
        torch.cuda.synchronize()
        timed3, mode3 = run_stack3, "eager launches"
        try:
            side = torch.cuda.Stream()
            side.wait_stream(torch.cuda.current_stream())
            with torch.cuda.stream(side):
                run_stack3()
            torch.cuda.current_stream().wait_stream(side)
            g3 = torch.cuda.CUDAGraph()
            with torch.cuda.graph(g3):
                run_stack3()
            g3.replay()
            torch.cuda.synchronize()
            if torch.equal(ref3, bufs3["down"]):
                timed3, mode3 = g3.replay, f"one HIP graph of {n_layers} layers, replayed"
        except Exception as exc:
            mode3 = f"eager launches (graph capture failed: {type(exc).__name__})"
        timed3()
        t3 = event_ms(timed3, 5, torch) / n_layers
        nbytes3 = sum(gemm_bytes(1, L3.K, L3.N) + 5 * L3.K for (L3, _, _) in protos3)
        decode[f"block_decode_{tag}"] = dict(M=1, layers=n_layers, us_per_layer=t3 * 1e3,
                                             us_per_token=t3 * 1e3 * n_layers,
                                             gbs=nbytes3 / (t3 * 1e-3) / 1e9, launch=mode3)
        del stack, protos3, bufs3, wss3


def main():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=50)
    ap.add_argument("--warmup", type=int, default=10)
    ap.add_argument("--no-cpu", action="store_true", help="skip the CPU-oracle baseline leg")
    ap.add_argument("--no-decode", action="store_true", help="skip the decode streaming leg")
    ap.add_argument("--no-train", action="store_true", help="skip the training-step leg")
    ap.add_argument("--no-prefill-30b", action="store_true",
                    help="skip the 30B layers at M = 4096 (they run the 6.7B step's GEMM kernel at another "
                         "size: a per-kernel profile of the step wants them out)")
    ap.add_argument("--no-decode-stacks", action="store_true",
                    help="decode leg: only the 30B-shaped launches (no 1.3B layer stream, no whole-block "
                         "steps): what a counter profile of those kernels wants")
    ap.add_argument("--cpu-seconds", type=float, default=15.0)
    ap.add_argument("--copy-calibration", action="store_true",
                    help="only run plain device copies of 256 MiB (reference for the rocprofv3 "
                         "FETCH_SIZE / WRITE_SIZE counters) and exit")
    args = ap.parse_args()
    if args.gpus != 1:
        print("bench.py measures one GPU: this build has no multi-GPU path (--gpus must be 1)",
              file=sys.stderr)
        sys.exit(2)

    import torch
    import paper_2310_11453_amd as bl

    bl.load_library()  # raises if the HIP library is missing: there is no fallback
    if not torch.cuda.is_available():
        raise SystemExit("bench.py needs a GPU")
    dev = torch.device("cuda:0")
    if args.copy_calibration:
        src = torch.empty(256 << 20, dtype=torch.uint8, device=dev).random_(0, 255)
        dst = torch.empty_like(src)
        for _ in range(10):
            dst.copy_(src)
        torch.cuda.synchronize()
        print(json.dumps({"copy_bytes_per_launch": src.numel(), "launches": 10}))
        return
    cfg = wl.CONFIGS[2]
    M = cfg.Ms[0]

    # ---- inputs: seeded, generated on the host, resident in HBM before timing ----------
    layers = []
    for li, L in enumerate(cfg.layers):
        seed = wl.seed_for(2, li)
        W = wl.make_weight(L.N, L.K, cfg.w_std, seed)
        X = wl.make_activation(M, L.K, seed, cfg.outlier_p, cfg.outlier_mul)
        Wd = torch.from_numpy(W).to(dev)
        packed, alpha, beta = bl.bitlinear_pack_weights(Wd)
        Xd = torch.from_numpy(X).to(dev)
        Y = torch.empty((M, L.N), dtype=torch.float32, device=dev)
        ws = torch.empty(bl.workspace_bytes(bl.OP_FORWARD, M, L.N, L.K), dtype=torch.uint8, device=dev)
        layers.append(dict(L=L, W=W, X=X, Wd=Wd, Xd=Xd, packed=packed, beta=beta, Y=Y, ws=ws))
    torch.cuda.synchronize()

    def step():
        for d in layers:
            bl.bitlinear_forward(d["Xd"], d["packed"], d["L"].N, d["beta"], out=d["Y"],
                                 workspace=d["ws"])

    # The GPU's clock takes some tens of milliseconds of load to settle (the same step measures
    # 292 us right after start and 262 us once it has): bring it there before the W warm-up steps,
    # so that short runs time the steady state too.  Untimed, like the warm-up.
    prewarm_steps = 150
    for _ in range(prewarm_steps + args.warmup):
        step()
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    ms_events = event_ms(step, args.steps, torch)
    torch.cuda.synchronize()
    ms_wall = (time.perf_counter() - t0) * 1e3 / args.steps
    ms_step = max(ms_events, 0.0)
    ops_step = sum(2 * M * d["L"].N * d["L"].K for d in layers)
    tops = ops_step / (ms_step * 1e-3) / 1e12

    # ---- per-kernel timing inside a second timed loop (events bracket each kernel) -------
    kern = {}
    for d in layers:
        L = d["L"]
        codes, gamma, rowsum, _ = bl.bitlinear_quant_act(d["Xd"])
        torch.cuda.synchronize()
        # the quantiser takes 10-35 us: timed from a graph of 20 launches (codes, gamma, row sums
        # into the layer's workspace, as bitlinear_forward does); the GEMM with events around
        # eager back-to-back launches (100+ us each: the queue never runs dry)
        qws = torch.empty(bl.workspace_bytes(bl.OP_QUANT, M, 1, L.K), dtype=torch.uint8, device=dev)
        lib = bl.load_library()

        def quant_once(i, d=d, L=L, codes=codes, gamma=gamma, rowsum=rowsum, qws=qws):
            rc = lib.bitlinear_quant_act(d["Xd"].data_ptr(), M, L.K, None, None, 1e-5, 0, 0,
                                         codes.data_ptr(), gamma.data_ptr(), rowsum.data_ptr(), None,
                                         qws.data_ptr(), qws.numel(),
                                         torch.cuda.current_stream().cuda_stream)
            assert rc == 0

        t_q, q_mode = graph_ms(quant_once, 20, max(2, args.steps // 10), torch)
        gemm_once = lambda: bl.bitlinear_matmul(codes, gamma, rowsum, d["packed"], L.N, d["beta"], out=d["Y"])
        for _ in range(100):  # back at the settled clock after the idle moments above
            gemm_once()
        t_g = event_ms(gemm_once, args.steps, torch)
        kern[L.name] = dict(quant_ms=t_q, quant_timing=q_mode, gemm_ms=t_g,
                            gemm_tops=2 * M * L.N * L.K / (t_g * 1e-3) / 1e12,
                            quant_gbs=5 * M * L.K / (t_q * 1e-3) / 1e9)
    up = layers[0]["L"]
    g_ms = kern[up.name]["gemm_ms"]
    roof = dict(bound="mfma", kernel="gemm_prefill_kernel<256,256,2,4,8> (4096->16384, M=2048)",
                achieved=2 * M * up.N * up.K / (g_ms * 1e-3) / 1e12, peak=I8_MFMA_PEAK_TOPS,
                unit="TOP/s", traffic=TRAFFIC_BYTES["gemm_prefill_up"], launch_ms=g_ms)
    roof["frac"] = roof["achieved"] / roof["peak"]

    # ---- weight preparation (Eq. 1-3, 12), once per weight at inference ----------------------
    d0 = layers[0]
    pws = torch.empty(bl.workspace_bytes(bl.OP_PACK, 0, up.N, up.K), dtype=torch.uint8, device=dev)
    t_pack = event_ms(lambda: bl.bitlinear_pack_weights(d0["Wd"], workspace=pws), 10, torch)
    prep = dict(ms=t_pack, gbs=(4 + 0.125) * up.N * up.K / (t_pack * 1e-3) / 1e9,
                note="one reading of fp32 W, and again the rows of tiles with a weight within |alpha| of zero")

    # ---- parity guard: a fast-but-wrong kernel must not report a number ----------------------
    # Both layers of the step: sampled rows of codes (given the normalised input the GPU dumped)
    # and sampled outputs of the timed launches against the oracle.
    import oracle
    ok = True
    signs, betas = [], []
    for d in layers:
        L = d["L"]
        codes, gamma, rowsum, xhat = bl.bitlinear_quant_act(d["Xd"], want_xhat=True)
        rows = np.arange(0, M, 257)
        xh = xhat[torch.from_numpy(rows).to(dev)].cpu().numpy()
        del xhat
        g_ref = oracle.absmax(xh)
        q_ref = oracle.quantize(xh, g_ref)
        ok = ok and np.array_equal(codes.cpu().numpy()[rows], q_ref)
        a, b = oracle.weight_stats(d["W"])
        sign = oracle.binarize(d["W"], a)
        signs.append(sign)
        betas.append(b)
        rng = np.random.default_rng(1)
        cols = rng.integers(0, L.N, rows.size * 16)
        rr = np.repeat(np.arange(rows.size), 16)
        acc = oracle.matmul_i32_sampled(q_ref, sign, rr, cols)
        y_ref = acc.astype(np.float32) * ((b * g_ref[rr]) / np.float32(128.0))
        y_gpu = d["Y"].cpu().numpy()[rows[rr], cols]
        ok = ok and np.array_equal(y_gpu, y_ref) and float(d["beta"].cpu()[0]) == float(b)
    parity = "ok" if ok else "FAILED"

    # ---- decode leg: packed-weight streaming on 30B-shaped layers, M = 16 and M = 1 ----------
    decode = None
    if not args.no_decode:
        decode = {"workload": "bitnet-30b layers, GEMM+dequant kernel per launch (prefill_30b: the same "
                              "layers at M = 4096, this leg holds their weights)", "shapes": []}
        c3 = wl.CONFIGS[3]
        best = None
        for li, L3 in enumerate(c3.layers):
            W3 = wl.make_weight(L3.N, L3.K, c3.w_std, wl.seed_for(3, li))
            p3, a3, b3 = bl.bitlinear_pack_weights(torch.from_numpy(W3).to(dev))
            # parity guard of this leg: 64 seeded output columns of every timed launch against the
            # oracle (from the GPU's own codes), all rows at M <= 64, 64 seeded rows at M = 4096
            a_ref, b_ref = oracle.weight_stats(W3)
            ns = np.sort(np.random.default_rng(li).choice(L3.N, 64, replace=False))
            sign_s = oracle.binarize(W3[ns], a_ref)
            del W3

            def sampled_ok(codes_t, gamma_t, Y_t, ms):
                q = codes_t[torch.from_numpy(ms).to(dev)].cpu().numpy()
                g = gamma_t.cpu().numpy()[ms]
                acc = oracle.matmul_i32(q, sign_s)
                y_ref = acc.astype(np.float32) * ((b_ref * g) / np.float32(128.0))[:, None]
                y = Y_t[torch.from_numpy(ms).to(dev)][:, torch.from_numpy(ns).to(dev)].cpu().numpy()
                return bool(np.array_equal(y, y_ref)) and float(b3.cpu()[0]) == float(b_ref)
            # rotate through copies so the working set (>= 512 MB) exceeds L2 + Infinity Cache
            ncopy = max(2, int(np.ceil(512e6 / p3.numel())))
            copies = [p3.clone() for _ in range(ncopy)]
            # The floor: a launch that only reads the same packed weights, with the small-batch
            # kernel's grid and loads (bitlinear_probe_read), over the same rotating copies.
            t_floor, _ = graph_ms(lambda i: bl.probe_read(copies[i % ncopy], 256, 448), 2 * ncopy, 5, torch)
            decode.setdefault("read_floor", []).append(
                dict(layer=L3.name, bytes=p3.numel(), us=t_floor * 1e3,
                     gbs=p3.numel() / (t_floor * 1e-3) / 1e9,
                     note="16-byte streaming loads of the packed weights only, 256 workgroups x 7 waves"))
            for Md in (1, 16, 64):  # M = 64 takes the MFMA-tile kernel: the ridge of the two rooflines
                X3 = torch.from_numpy(wl.make_activation(Md, L3.K, wl.seed_for(3, li))).to(dev)
                codes3, gamma3, rowsum3, _ = bl.bitlinear_quant_act(X3)
                Y3 = torch.empty((Md, L3.N), dtype=torch.float32, device=dev)
                ws3 = torch.empty(max(256, bl.workspace_bytes(bl.OP_MATMUL, Md, L3.N, L3.K)),
                                  dtype=torch.uint8, device=dev)

                def run(i):
                    bl.bitlinear_matmul(codes3, gamma3, rowsum3, copies[i % ncopy], L3.N,
                                        b3, out=Y3, workspace=ws3)

                t, t_mode = graph_ms(run, 2 * ncopy, 5, torch)
                if not sampled_ok(codes3, gamma3, Y3, np.arange(Md)):
                    parity = "FAILED"
                gbs = gemm_bytes(Md, L3.K, L3.N) / (t * 1e-3) / 1e9
                tops3 = 2 * Md * L3.K * L3.N / (t * 1e-3) / 1e12
                rec = dict(layer=L3.name, K=L3.K, N=L3.N, M=Md, us=t * 1e3, gbs=gbs,
                           frac_hbm=gbs / HBM_PEAK_GBS, tops=tops3,
                           frac_i8_mfma_peak=tops3 / I8_MFMA_PEAK_TOPS,
                           x_read_floor=t / t_floor, timing=t_mode)
                decode["shapes"].append(rec)
                if Md <= 16 and (best is None or gbs > best["gbs"]):
                    best = rec
            del copies
            # the same layer at the configuration's prefill batch (M = 4096): GEMM + dequant launch
            # alone, after enough launches for the clock to settle
            if args.no_prefill_30b:
                del p3
                continue
            Mp = 4096
            Xp = torch.from_numpy(wl.make_activation(Mp, L3.K, wl.seed_for(3, 20 + li))).to(dev)
            cp, gp, rp, _ = bl.bitlinear_quant_act(Xp)
            del Xp
            Yp = torch.empty((Mp, L3.N), dtype=torch.float32, device=dev)

            def run_p():
                bl.bitlinear_matmul(cp, gp, rp, p3, L3.N, b3, out=Yp)

            for _ in range(100):
                run_p()
            tp = event_ms(run_p, 30, torch)
            if not sampled_ok(cp, gp, Yp, np.sort(np.random.default_rng(7 + li).choice(Mp, 64, replace=False))):
                parity = "FAILED"
            tops_p = 2 * Mp * L3.K * L3.N / (tp * 1e-3) / 1e12
            decode.setdefault("prefill_30b", []).append(
                dict(layer=L3.name, K=L3.K, N=L3.N, M=Mp, us=tp * 1e3, tops=tops_p,
                     frac_i8_mfma_peak=tops_p / I8_MFMA_PEAK_TOPS))
            del cp, Yp, p3

        # Group Quantization and Normalization (Eq. 13-15) at a 30B shape, eight groups on each axis:
        # what a tensor-parallel layer computes, all shards on this one GPU: the quantiser on the K-slices,
        # then one GEMM launch that walks all K-groups and writes Y once.
        Lg, G = c3.layers[1], 8
        Wg = wl.make_weight(Lg.N, Lg.K, c3.w_std, wl.seed_for(3, 30))
        pg, ag, bg = bl.bitlinear_pack_weights_grouped(torch.from_numpy(Wg).to(dev), G, G)
        del Wg
        grouped = []
        for Mg in (16, 4096):
            Xg = torch.from_numpy(wl.make_activation(Mg, Lg.K, wl.seed_for(3, 31))).to(dev)
            Yg = torch.empty((Mg, Lg.N), dtype=torch.float32, device=dev)
            fg = lambda: bl.bitlinear_forward_grouped(Xg, pg, Lg.N, bg, G, G, out=Yg)
            for _ in range(20):
                fg()
            if Mg <= 64:
                tg, how = graph_ms(lambda i: fg(), 20, 10, torch)
            else:
                tg, how = event_ms(fg, 20, torch), "HIP events"
            grouped.append(dict(layer=Lg.name, K=Lg.K, N=Lg.N, M=Mg, groups_n=G, groups_k=G, us=tg * 1e3,
                                tops=2 * Mg * Lg.K * Lg.N / (tg * 1e-3) / 1e12, timing=how,
                                note="LN + quantiser per K-group, then all K-groups in one GEMM launch"))
            del Xg, Yg
        decode["grouped_30b"] = grouped
        del pg
        if not args.no_decode_stacks:
            decode_stacks(bl, torch, dev, decode)
        decode["value"] = best["gbs"]
        decode["unit"] = "GB/s"
        decode["roofline"] = dict(bound="hbm", kernel="gemm_decode_kernel", achieved=best["gbs"],
                                  peak=HBM_PEAK_GBS, unit="GB/s", frac=best["gbs"] / HBM_PEAK_GBS,
                                  traffic=None,
                                  note="launches replayed back to back from one HIP graph over rotating "
                                       "weight copies; read_floor is the same bytes only read")

    # ---- training-step leg: forward + STE backward (Section 2.2) at M = 8192, 4096 -> 16384 ----
    # Weights change every step, so the step starts from fp32 W: pack (Eq. 1-3), forward
    # (Eq. 12, 4-5, 7, 11), dX^ and dW by the straight-through estimator, dx through LayerNorm.
    train = None
    if not args.no_train:
        c4 = wl.CONFIGS[4]
        L4, M4 = c4.layers[0], c4.Ms[0]
        s4 = wl.seed_for(4, 0)
        W4 = torch.from_numpy(wl.make_weight(L4.N, L4.K, c4.w_std, s4)).to(dev)
        X4 = torch.from_numpy(wl.make_activation(M4, L4.K, s4)).to(dev)
        dY4 = torch.from_numpy(wl.make_grad(M4, L4.N, s4)).to(dev)
        Y4 = torch.empty((M4, L4.N), dtype=torch.float32, device=dev)
        wsb = torch.empty(bl.workspace_bytes(bl.OP_BACKWARD, M4, L4.N, L4.K, True),
                          dtype=torch.uint8, device=dev)
        st4 = {}

        def t_pack():
            st4["packed"], _, st4["beta"] = bl.bitlinear_pack_weights(W4, workspace=pws)

        def t_fwd():
            st4["q"] = bl.bitlinear_quant_act(X4, per_tensor=True)
            bl.bitlinear_matmul(st4["q"][0], st4["q"][1], st4["q"][2], st4["packed"], L4.N,
                                st4["beta"], per_tensor=True, out=Y4)

        def t_bwd():
            st4["dX"], st4["dW"] = bl.bitlinear_backward_ste(
                dY4, st4["q"][0], st4["q"][1], st4["packed"], st4["beta"], True, workspace=wsb)

        def t_ln():
            bl.bitlinear_layernorm_backward(st4["dX"], X4, out=st4["dX"])

        def t_all():
            t_pack(), t_fwd(), t_bwd(), t_ln()

        t_all()
        torch.cuda.synchronize()
        parts = {n: event_ms(f, 5, torch) for n, f in
                 (("pack_ms", t_pack), ("forward_ms", t_fwd), ("backward_ste_ms", t_bwd),
                  ("ln_backward_ms", t_ln), ("step_ms", t_all))}
        fl = 2.0 * M4 * L4.N * L4.K
        train = dict(workload=f"train-step: M={M4}, {L4.K}->{L4.N}, per-tensor gamma, dY~N(0,1e-6)",
                     **parts, forward_tops=fl / (parts["forward_ms"] * 1e-3) / 1e12,
                     backward_tflops=2 * fl / (parts["backward_ste_ms"] * 1e-3) / 1e12,
                     backward_frac_bf16_peak=2 * fl / (parts["backward_ste_ms"] * 1e-3) / 1e12 / 2500.0,
                     note="backward_ste = one pass over dY (bf16 copies), bit expansion, code "
                          "transpose, two bf16 MFMA GEMMs")
        del W4, X4, dY4, Y4, wsb, st4

    # ---- CPU oracle on a bounded sample of the same workload ---------------------------------
    # The same step (LN, quantise, integer GEMM, dequant through both layers) on the first
    # s_rows tokens, repeated `reps` times, sized from a small calibration run to about
    # --cpu-seconds of work.  Binarising the weights is outside the timed region, as packing is
    # on the GPU.
    cpu = None
    if not args.no_cpu:
        threads = oracle.num_threads()
        per_row = 0.0
        for d, sg in zip(layers, signs):
            xh = oracle.layernorm(d["X"][:8])
            q = oracle.quantize(xh, oracle.absmax(xh))
            oracle.matmul_i32(q, sg[:2048])
            t0 = time.perf_counter()
            oracle.matmul_i32(q, sg[:2048])
            per_row += max(time.perf_counter() - t0, 1e-4) / 8 * (d["L"].N / 2048)
        s_rows = int(min(M, max(8, args.cpu_seconds / per_row)))

        def cpu_step():
            for d, sg, b_l in zip(layers, signs, betas):
                xh = oracle.layernorm(d["X"][:s_rows])
                g = oracle.absmax(xh)
                q = oracle.quantize(xh, g)
                acc = oracle.matmul_i32(q, sg)
                oracle.dequant(acc, g, b_l)

        t0 = time.perf_counter()
        cpu_step()
        dt = time.perf_counter() - t0
        reps = 1
        extra = int(args.cpu_seconds / dt) - 1  # the calibration above overestimates: fill the budget
        if extra > 0:
            for _ in range(extra):
                cpu_step()
            reps += extra
            dt = time.perf_counter() - t0
        ops = reps * sum(2 * s_rows * d["L"].N * d["L"].K for d in layers)
        cpu = dict(value=ops / dt / 1e12, unit="TOPS", cores=threads, kind="oracle", seconds=dt,
                   sample=f"{reps} x the step on the first {s_rows} of {M} tokens (LN, quantise, "
                          f"int GEMM, dequant through both layers); weights pre-binarised")

    # ---- analytic arithmetic energy of the step's products (Section 3's estimate; context only) ----
    from paper_2310_11453_amd import energy as en
    e_bit = [en.bitlinear_energy(M, d["L"].K, d["L"].N, "7nm") for d in layers]
    e_f16 = [en.matmul_energy(M, d["L"].K, d["L"].N, "fp16", "7nm") for d in layers]
    energy_model = dict(node="7nm", unit="J per step", bitlinear_add=sum(e[0] for e in e_bit),
                        bitlinear_mul=sum(e[1] for e in e_bit), fp16_add=sum(e[0] for e in e_f16),
                        fp16_mul=sum(e[1] for e in e_f16),
                        note="the paper's per-operation energy model applied to the two products of "
                             "the step; not a measurement")

    out = {
        "metric": "BitLinear prefill TOPS (i8 MFMA %) + decode packed-weight HBM GB/s",
        "value": tops, "unit": "TOPS", "n_gpus": 1, "steps": args.steps, "warmup": args.warmup,
        "ms_per_step": ms_step, "ms_per_step_wall": ms_wall, "prewarm_steps": prewarm_steps, "higher_is_better": True,
        "scaling": "weak", "vs_baseline": None, "dtype": "i8 x 1-bit -> i32, f32 out",
        "data": "synthetic",
        "config": {"workload": "bitnet-6.7b-prefill: BitLinear forward 4096->16384 and "
                               "16384->4096, M=2048, per-token gamma, fp32 in/out",
                   "step": "LN+quantise+GEMM+dequant for both layers; weights packed beforehand"},
        "mfma_frac_of_peak": tops / I8_MFMA_PEAK_TOPS,
        "kernels": kern, "roofline": roof, "weight_prep": prep, "decode": decode, "training": train, "energy_model": energy_model,
        "cpu_baseline": cpu, "parity": parity,
    }
    if parity != "ok":  # no number without parity
        for key in ("value", "mfma_frac_of_peak"):
            out[key] = None
        out["roofline"] = dict(out["roofline"], achieved=None, frac=None)
        print(json.dumps(out))
        sys.exit(1)
    print(json.dumps(out))


if __name__ == "__main__":
    main()
