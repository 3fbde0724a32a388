"""Benchmark: one "step" = one pass of the whole hot path (plan lookup, Image-halo and Filter staging, MFMA
contraction, Out epilogue: one cacnn_conv_forward call) over one batch of synthetic input resident in HBM.

Prints ONE JSON line.  metric/unit follow the benchmark definition (conv TFLOP/s on one MI355X); the headline
workload is c5, the largest of the five shapes; `roofline` prices the kernel against the MFMA peak of its dtype;
`cpu_baseline` is the fp64 loop-nest oracle timed on the host in the same run; `shapes` carries the same
measurements for all five benchmark shapes.

Order of the run: every input is generated and uploaded first; then the machine's sustained rates are measured
(register-only MFMA loops and a streaming copy); then, per shape: about 0.3 s of the register-only MFMA loop of the
shape's dtype (power-state conditioning: the board's power management needs a few hundred milliseconds of matrix load
to settle, and a cold chip runs the first launches of c5 up to 25 % slower, see profiles/clock_ramp_c2_c5.txt), then the W
warm-up launches, then exactly K timed launches between two events on the launch stream.
"""
import argparse
import json
import os
import re
import sys
import time

ROOT = os.path.dirname(os.path.abspath(__file__))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)

MFMA_PEAK_TFLOPS = {"f32": 157.3, "bf16": 2500.0}      # MI355X published dense MFMA peaks
HBM_PEAK_GBS = 8000.0
LDS_BYTES = 160 * 1024


def upload_config(torch, ci, np, cfg):
    """Seeded host inputs and their device copies (bf16 as raw 16-bit patterns), plus the Out buffer."""
    img, flt = ci.make_inputs(cfg)
    if cfg.dtype == "bf16":
        d_img = torch.from_numpy(ci.bf16_bits(img).view(np.int16).reshape(-1)).cuda()
        d_flt = torch.from_numpy(ci.bf16_bits(flt).view(np.int16).reshape(-1)).cuda()
    else:
        d_img = torch.from_numpy(img.reshape(-1)).cuda()
        d_flt = torch.from_numpy(flt.reshape(-1)).cuda()
    d_out = torch.empty(int(np.prod(cfg.out_shape)), dtype=torch.float32, device="cuda:0")
    return img, flt, d_img, d_flt, d_out


_COND = {}


def condition_power_state(cc, torch, ci, np, dtype, ms=300.0):
    """About `ms` milliseconds of the register-only MFMA loop of this dtype on every compute unit: brings the board's
    power management to the state a steady matrix load runs in.  Untimed; no workload kernel runs in it."""
    dt = 0 if dtype == "f32" else 1
    if dt not in _COND:
        rng = np.random.default_rng(18020690)
        if dt == 0:
            words = rng.uniform(-1.0, 1.0, 4096).astype(np.float32).view(np.int32)
        else:
            words = np.ascontiguousarray(
                ci.bf16_bits(ci.round_to_bf16(rng.standard_normal(8192).astype(np.float32)))).view(np.int32)
        _COND[dt] = (torch.from_numpy(np.ascontiguousarray(words)).cuda(),
                     torch.empty(65536, dtype=torch.float32, device="cuda:0"))
    ops, sink = _COND[dt]
    t0 = time.perf_counter()
    while (time.perf_counter() - t0) * 1e3 < ms:
        cc.cacnn_probe_mfma(dt, ops, sink, 800 if dt == 0 else 1600)
        torch.cuda.synchronize()


def time_config(cc, torch, ci, np, cfg, steps, warmup, buffers, repeats=1, condition=True):
    """Average launch duration (seconds) of cacnn_conv_forward over `steps` back-to-back launches, measured with
    events on the stream the kernel runs on (torch's current stream)."""
    img, flt, d_img, d_flt, d_out = buffers
    dt = 0 if cfg.dtype == "f32" else 1
    if condition:
        condition_power_state(cc, torch, ci, np, cfg.dtype)
    for _ in range(warmup):
        cc.cacnn_conv_forward(cfg.dims, dt, d_img, d_flt, d_out)
    best = None
    for _ in range(repeats):
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        t0 = time.perf_counter()
        e0.record()
        for _ in range(steps):
            cc.cacnn_conv_forward(cfg.dims, dt, d_img, d_flt, d_out)
        e1.record()
        torch.cuda.synchronize()
        wall = time.perf_counter() - t0
        ev = e0.elapsed_time(e1) * 1e-3
        if best is None or ev < best[0]:
            best = (ev, wall)
    return best[0] / steps, best[1] / steps


def machine_sustained(cc, torch, ci, np):
    """What this machine sustains, measured now: a register-only MFMA loop on every CU (operands with the value mix of the
    workloads, and all-zero operands, which toggle nothing and let the clock stay high) and a 1 GiB streaming copy.
    The published peaks assume 2.4 GHz; an all-CU matrix load is power-managed below that."""
    def timed(fn, warm, reps):
        for _ in range(warm):
            fn()
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        torch.cuda.synchronize()
        e0.record()
        for _ in range(reps):
            fn()
        e1.record()
        torch.cuda.synchronize()
        return e0.elapsed_time(e1) * 1e-3 / reps
    rng = np.random.default_rng(18020690)
    sink = torch.empty(65536, dtype=torch.float32, device="cuda:0")
    out = {}
    for name, dt, flops, iters in (("f32", 0, 4096.0, 800), ("bf16", 1, 32768.0, 1600)):
        if dt == 0:
            words = rng.uniform(-1.0, 1.0, 4096).astype(np.float32).view(np.int32)
        else:
            words = np.ascontiguousarray(ci.bf16_bits(ci.round_to_bf16(rng.standard_normal(8192).astype(np.float32)))).view(np.int32)
        for label, host in (("", words), ("_zero_operands", np.zeros(4096, dtype=np.int32))):
            ops = torch.from_numpy(np.ascontiguousarray(host)).cuda()
            n = [0]
            def launch():
                n[0] = cc.cacnn_probe_mfma(dt, ops, sink, iters)
            sec = timed(launch, 30, 30)
            out[f"mfma_{name}_tflops{label}"] = n[0] * flops / sec / 1e12
    nbytes = 1 << 30
    src = torch.empty(nbytes, dtype=torch.uint8, device="cuda:0").fill_(1)
    dst = torch.empty(nbytes, dtype=torch.uint8, device="cuda:0")
    sec = timed(lambda: cc.cacnn_probe_copy(src, dst, nbytes), 5, 10)
    out["copy_GBps_read_plus_write"] = 2.0 * nbytes / sec / 1e9
    # every CU filling its LDS with the staging waves' loads: from a window one L2 holds, and from one far beyond the L2s
    for label, window in (("l2_to_lds_GBps", 2 << 20), ("beyond_l2_to_lds_GBps", 512 << 20)):
        moved = [0]
        def fill():
            moved[0] = cc.cacnn_probe_lds_fill(src, window, sink, 400)
        sec = timed(fill, 3, 10)
        out[label] = moved[0] / sec / 1e9
    # the bf16 convolution's unit with nothing that synchronises its two halves: per compute unit and iteration 4 x 42
    # MFMAs (1344 MFMA cycles per SIMD) and 48 KiB from the L2 into the LDS; alone, and side by side
    words = np.ascontiguousarray(ci.bf16_bits(ci.round_to_bf16(rng.standard_normal(8192).astype(np.float32)))).view(np.int32)
    ops = torch.from_numpy(np.ascontiguousarray(words)).cuda()
    n = 2000
    for label, (mi, fi) in (("unit_mix_mfma_alone_ns", (n, 0)), ("unit_mix_fill_alone_ns", (0, n)),
                            ("unit_mix_side_by_side_ns", (n, n)),
                            # c4's unit: 24 MFMAs per wave and 45 KiB, i.e. 2000 of them are 1143 x 42 MFMAs and 1875 x 48 KiB
                            ("unit_mix_c4_side_by_side_ns", (1143, 1875)),
                            # the same MFMAs with the bytes two other tilings of c4 would stage per unit: an Image unit that
                            # serves all three filter rows (33.9 KiB per 24 MFMAs), 128 output channels x half the positions
                            # (41 KiB)
                            ("unit_mix_c4_three_rows_per_image_unit_ns", (1143, 1412)),
                            ("unit_mix_c4_k128_half_positions_ns", (1143, 1708)),
                            ("unit_mix_c4_mfma_alone_ns", (1143, 0))):
        sec = timed(lambda: cc.cacnn_probe_mfma_and_fill(ops, src, 2 << 20, sink, mi, fi), 3, 10)
        out[label] = sec / n * 1e9
    # the same mixes on as many compute units as the two bf16 shapes have tiles (the others idle), and on half of them:
    # how a unit's time depends on how many compute units work at once; and with the MFMA waves reading their operands
    # from the LDS being filled (a window of N(0,1) bf16 words, so that the operands toggle as the register-only loop's do)
    win = torch.from_numpy(np.ascontiguousarray(ci.bf16_bits(ci.round_to_bf16(rng.standard_normal(1 << 20).astype(np.float32)))
                                                .view(np.int16))).cuda()
    for label, cus, tile, reads, (mi, fi) in (("unit_mix_side_by_side_224_cus_ns", 224, 0, 0, (n, n)),
                                              ("unit_mix_side_by_side_128_cus_ns", 128, 0, 0, (n, n)),
                                              ("unit_mix_mfma_alone_224_cus_ns", 224, 0, 0, (n, 0)),
                                              ("unit_mix_mfma_alone_128_cus_ns", 128, 0, 0, (n, 0)),
                                              ("unit_mix_with_lds_reads_224_cus_ns", 224, 0, 1, (n, n)),
                                              ("unit_mix_with_lds_reads_256_cus_ns", 256, 0, 1, (n, n)),
                                              ("unit_mix_mfma_with_lds_reads_no_fill_224_cus_ns", 224, 0, 1, (n, 0)),
                                              ("unit_mix_c4_side_by_side_196_cus_ns", 196, 0, 0, (1143, 1875)),
                                              ("unit_mix_c4_side_by_side_128_cus_ns", 128, 0, 0, (1143, 1875)),
                                              # c4's own MFMA loop (24 MFMAs per wave and iteration on 4 accumulators)
                                              ("unit_mix_c4_own_loop_mfma_alone_196_cus_ns", 196, 1, 0, (n, 0)),
                                              ("unit_mix_c4_own_loop_side_by_side_196_cus_ns", 196, 1, 0, (n, 1875)),
                                              ("unit_mix_c4_own_loop_with_lds_reads_no_fill_196_cus_ns", 196, 1, 1, (n, 0)),
                                              ("unit_mix_c4_with_lds_reads_196_cus_ns", 196, 1, 1, (n, 1875)),
                                              ("unit_mix_c4_with_lds_reads_256_cus_ns", 256, 1, 1, (n, 1875)),
                                              # with a workgroup barrier per unit as well (mode 3; the c4 unit then with 48
                                              # instead of 45 KiB: the barrier needs equal iteration counts)
                                              ("unit_mix_with_lds_reads_and_barrier_224_cus_ns", 224, 0, 3, (n, n)),
                                              ("unit_mix_c4_with_lds_reads_48k_196_cus_ns", 196, 1, 1, (n, n)),
                                              ("unit_mix_c4_with_lds_reads_48k_and_barrier_196_cus_ns", 196, 1, 3, (n, n))):
        sec = timed(lambda: cc.cacnn_probe_mfma_and_fill_on(cus, tile, reads, ops, win, 2 << 20, sink, mi, fi), 3, 10)
        out[label] = sec / n * 1e9
    del src, dst
    return out


def graph_replay_us(cc, torch, ci, np, cfg, buffers, launches=200, replays=20):
    """Per-launch time of the workload when `launches` back-to-back launches are captured in one HIP graph and replayed:
    what a launch-bound caller gets (the plain figure is bound by the host's launch path for a problem as small as c1)."""
    _, _, d_img, d_flt, d_out = buffers
    dt = 0 if cfg.dtype == "f32" else 1
    cc.cacnn_conv_forward(cfg.dims, dt, d_img, d_flt, d_out)     # plan and kernel set-up happen outside the capture
    torch.cuda.synchronize()
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.stream(side):
        with torch.cuda.graph(graph, stream=side):
            for _ in range(launches):
                cc.cacnn_conv_forward(cfg.dims, dt, d_img, d_flt, d_out)
    torch.cuda.synchronize()
    for _ in range(3):
        graph.replay()
    e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    torch.cuda.synchronize()
    e0.record()
    for _ in range(replays):
        graph.replay()
    e1.record()
    torch.cuda.synchronize()
    return e0.elapsed_time(e1) * 1e3 / (replays * launches)


def committed_traffic(name, variant=None, xcd_split_k=None):
    """HBM-side bytes of one launch from the committed rocprofv3 --pmc summary (FETCH_SIZE and WRITE_SIZE runs, scaled
    by the copy-kernel calibration recorded there).  Counters cannot be read from inside this process, so the figure is
    the one RECORDED for this shape, not a measurement of this run.  Each `traffic` row names the kernel variant and the
    XCD division it was recorded with; if the plan of this run differs (or the row names none), the figure would
    belong to another launch configuration and None is returned instead."""
    for fname in ("hbm_traffic_c1-c5.txt", "pooling_p1.txt", "two_level_layouts.txt"):
        try:
            with open(os.path.join(ROOT, "profiles", fname)) as f:
                for line in f:
                    t = line.split()
                    if len(t) >= 5 and t[0] == "traffic" and t[1] == name:
                        if variant is not None:
                            rec = line.split("|")
                            if len(rec) < 3 or rec[1].strip() != variant or int(rec[2].split()[0]) != int(xcd_split_k):
                                return None
                        return float(t[4])
        except (OSError, ValueError):
            pass
    return None


def shape_report(cc, cfg, sec):
    dt = 0 if cfg.dtype == "f32" else 1
    esz = 4 if dt == 0 else 2
    flops = 2.0 * cfg.macs
    tflops = flops / sec / 1e12
    plan = cc.cacnn_tile_plan(cfg.dims, dt)
    n_img = 1
    for x in cfg.image_shape:
        n_img *= x
    n_flt = cfg.K * cfg.R * cfg.S * cfg.C
    n_out = cfg.K * cfg.H * cfg.W * cfg.B
    compulsory = esz * (n_img + n_flt) + 4 * n_out
    def bound_bytes(fast_bytes):
        b = cc.cacnn_lower_bound(cfg.dims, fast_bytes / esz)
        return max(4 * b.term[0], esz * max(b.term[1:]))
    lb_bytes = bound_bytes(LDS_BYTES)
    # what was timed: the planned variant, or a kernel with flattened positions, which no plan describes
    vname, grid, _ = cc.binding.routed_kernel(cfg.dims, dt)
    planned = vname == cc.cacnn_variant_name(plan.variant)
    hbm = committed_traffic(cfg.name, vname, plan.xcd_split_k if planned else 0)
    F = float(cfg.macs)
    M_lds = LDS_BYTES / esz
    staged = esz * (plan.predicted_words - n_out) + 4 * n_out if planned else None

    def xcd_level_bound_bytes():
        # Two levels: an LDS tile inside an XCD's share.  The HBM-side bytes are the misses of eight 4 MiB L2s, so the
        # bound that applies to them is Section 7's (eight processors, M = one L2) for the division the launch uses:
        # a_K groups of output channels x 8 / a_K ranges of positions (only the product a_B a_W a_H enters the bound)
        ak = max(1, plan.xcd_split_k) if planned else 1
        rest, a = 8 // ak, [1, ak, 1, 1]
        for i, extent in ((0, cfg.B), (3, cfg.H), (2, cfg.W)):
            f = 1
            while f * 2 <= min(rest, extent):
                f *= 2
            a[i], rest = f, rest // f
        b = cc.cacnn_parallel_bound(cfg.dims, 4 * 1024 * 1024 / esz, a)
        return max(4 * b.term[0], esz * max(b.term[1:])), a
    xcd_bound, xcd_div = xcd_level_bound_bytes()
    return {
        "us": sec * 1e6, "tflops": tflops, "frac_mfma_peak": tflops / MFMA_PEAK_TFLOPS[cfg.dtype],
        "frac_hbm_roofline": compulsory / sec / 1e9 / HBM_PEAK_GBS,
        "compulsory_bytes": compulsory, "paper_bound_bytes_at_M_lds": lb_bytes,
        # the same bound with a CU's registers counted as fast memory too, and with one XCD's 4 MiB L2 as the fast
        # memory (the level whose misses the profiled HBM-side bytes are)
        "paper_bound_bytes_at_M_lds_plus_vgpr": bound_bytes(LDS_BYTES + 512 * 1024),
        "paper_bound_bytes_at_M_l2": bound_bytes(4 * 1024 * 1024),
        "hbm_bytes_over_bound_at_M_lds": (hbm / lb_bytes) if hbm else None,
        "hbm_bytes_over_bound_at_M_l2": (hbm / bound_bytes(4 * 1024 * 1024)) if hbm else None,
        "xcd_division_a_B_a_K_a_W_a_H": xcd_div, "paper_parallel_bound_bytes_8_xcds_M_l2": xcd_bound,
        "hbm_bytes_over_parallel_bound": (hbm / xcd_bound) if hbm else None,
        # global -> LDS bytes of the launched schedule plus Out once (cacnn_plan.predicted_words, in bytes): the traffic
        # the paper's model counts at M = LDS, against Theorem 1 and against matmul-style reuse F / sqrt(M) (Section 1); none for a
        # kernel with flattened positions
        "planned_staged_bytes": staged,
        "staged_bytes_over_bound_at_M_lds": staged / lb_bytes if planned else None,
        "matmul_reuse_bytes_at_M_lds": esz * F / M_lds ** 0.5,
        "staged_bytes_over_matmul_reuse": staged / (esz * F / M_lds ** 0.5) if planned else None,
        "variant": vname, "grid": grid, "lds_bytes": plan.lds_bytes_used if planned else None,
        "b_c": plan.b_c if planned else None, "hbm_bytes_recorded": hbm,
    }


def alternative_variants_us(cc, torch, cfg, buffers, steps, warmup):
    """Launch time of every OTHER fixed-geometry kernel variant that accepts the shape (same process, same buffers, right
    after the planner's own variant was timed): the evidence for the planner's choice among them."""
    _, _, d_img, d_flt, d_out = buffers
    dt = 0 if cfg.dtype == "f32" else 1
    chosen = cc.cacnn_tile_plan(cfg.dims, dt)
    out = {}
    for vi in range(cc.cacnn_variant_count()):
        name = cc.cacnn_variant_name(vi)
        if vi == chosen.variant or " fx" not in name or not name.startswith(cfg.dtype + " "):
            continue
        ct, br, bs = re.search(r" c(\d+)r(\d+)s(\d+)", name).groups()       # ... c32r3s1 [s2 | t8]
        plan = cc.cacnn_tile_plan(cfg.dims, dt)
        plan.variant, plan.b_c, plan.b_r, plan.b_s = vi, int(ct), int(br), int(bs)
        plan.xcd_split_k = 0
        try:
            for _ in range(warmup):
                cc.cacnn_conv_forward_with_plan(cfg.dims, dt, plan, d_img, d_flt, d_out)
        except cc.CacnnError:
            continue                                                        # the variant does not take this shape
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        e0.record()
        for _ in range(steps):
            cc.cacnn_conv_forward_with_plan(cfg.dims, dt, plan, d_img, d_flt, d_out)
        e1.record()
        torch.cuda.synchronize()
        out[name] = e0.elapsed_time(e1) * 1e3 / steps
    return out


def add_unit_mix(rep, cfg, sustained):
    """For c4 and c5: the units a workgroup runs (Out tiles per workgroup x c-slices x filter rows) times what the machine
    takes for one unit's MFMAs and bytes side by side with nothing synchronising them, on as many compute units as the
    shape has tiles (machine_sustained; with the operands read from the LDS as the shape's kernel reads them): the time
    the launch's loop would take at that rate, without the start and the end of a launch."""
    key = {"c5": "unit_mix_with_lds_reads_224_cus_ns", "c4": "unit_mix_c4_with_lds_reads_196_cus_ns"}.get(cfg.name)
    if key is None or key not in sustained:
        return
    units = (cfg.C // 32) * cfg.S            # one tile per workgroup on both shapes
    rep["units_per_workgroup"] = units
    rep["loop_us_at_unsynchronised_mix_rate"] = units * sustained[key] * 1e-3


def cpu_baseline(cfg, img, flt, np):
    """The oracle as it stands, all host threads, on the whole workload when that is a few seconds of CPU work,
    otherwise on the first k output channels (the work per channel is identical)."""
    from oracle import conv as oconv
    threads = oconv.num_threads()
    K = cfg.K
    budget_macs = 40e9          # about 10-30 s on a few cores
    k_use = max(1, min(K, int(K * budget_macs / cfg.macs)))
    p = oconv.Problem(cfg.B, cfg.C, k_use, cfg.W, cfg.H, cfg.R, cfg.S, cfg.sigma_w, cfg.sigma_h)
    sub = np.ascontiguousarray(flt[:k_use])
    oconv.conv_fp64(oconv.Problem(cfg.B, cfg.C, 1, cfg.W, cfg.H, cfg.R, cfg.S, cfg.sigma_w, cfg.sigma_h), img,
                    np.ascontiguousarray(flt[:1]))            # load the library, touch the inputs
    # repeat the sample until about ten seconds of host work have been timed (a single pass of the small shapes is
    # too short to time well)
    reps, total = 0, 0.0
    while total < 10.0 and reps < 1000:
        t0 = time.perf_counter()
        ref, ab = oconv.conv_fp64(p, img, sub)
        total += time.perf_counter() - t0
        reps += 1
    dt = total / reps
    macs = cfg.macs * k_use / K
    return {"value": 2.0 * macs / dt / 1e12, "unit": "TFLOP/s", "cores": threads, "kind": "oracle",
            "sample": f"{cfg.name}: output channels 0..{k_use - 1} of {K} ({macs:.3g} MACs, fp64, {dt:.3f} s per pass, "
                      f"{reps} passes)"}, ref, ab, k_use


def traffic_probe(cc, torch, ci, np, cfg, xcd_split_k=0, xcd_walk=0):
    """Dispatch sequence for the HBM-traffic counters (FETCH_SIZE / WRITE_SIZE, KiB per dispatch):
    a plain copy of known size to scale the counters by, then the workload cold (caches evicted) and warm.
    xcd_split_k > 0 forces that division of the XCDs over the output channels on the planned variant (0: what cacnn_conv_forward runs)."""
    n = 512 * 1024 * 1024
    src = torch.empty(n, dtype=torch.uint8, device="cuda:0").fill_(1)
    dst = torch.empty(n, dtype=torch.uint8, device="cuda:0")
    img, flt = ci.make_inputs(cfg)
    if cfg.dtype == "bf16":
        d_img = torch.from_numpy(ci.bf16_bits(img).view(np.int16).reshape(-1)).cuda()
        d_flt = torch.from_numpy(ci.bf16_bits(flt).view(np.int16).reshape(-1)).cuda()
    else:
        d_img = torch.from_numpy(img.reshape(-1)).cuda()
        d_flt = torch.from_numpy(flt.reshape(-1)).cuda()
    d_out = torch.empty(int(np.prod(cfg.out_shape)), dtype=torch.float32, device="cuda:0")
    dt = 0 if cfg.dtype == "f32" else 1
    torch.cuda.synchronize()
    dst.copy_(src)                                   # calibration: reads n bytes, writes n bytes
    torch.cuda.synchronize()
    evict = torch.empty(1024 * 1024 * 1024, dtype=torch.uint8, device="cuda:0").fill_(3)   # push everything out
    torch.cuda.synchronize()
    plan = cc.cacnn_tile_plan(cfg.dims, dt)
    variant = cc.cacnn_variant_name(plan.variant)
    if xcd_split_k:
        plan.xcd_split_k, plan.xcd_walk = xcd_split_k, xcd_walk
    elif cc.binding.routed_kernel(cfg.dims, dt)[0] != variant:
        variant, plan.xcd_split_k, plan.xcd_walk = cc.binding.routed_kernel(cfg.dims, dt)[0], 0, 0
    for _ in ("cold", "warm"):
        if plan.xcd_split_k:
            cc.cacnn_conv_forward_with_plan(cfg.dims, dt, plan, d_img, d_flt, d_out)
        else:
            cc.cacnn_conv_forward(cfg.dims, dt, d_img, d_flt, d_out)
        torch.cuda.synchronize()
    del evict
    print(json.dumps({"traffic_probe": cfg.name, "copy_bytes_each_way": n, "xcd_split_k": plan.xcd_split_k,
                      "xcd_walk": plan.xcd_walk, "variant": variant}))


def division_report(cc, torch, ci, np, cfg, steps, warmup):
    """Two levels, the eight XCDs as Section 7's processors: for every layout of an XCD's run of tiles that
    cacnn_two_level_plan considers (a_K groups of output channels x the order inside a group), the time of the workload, the
    words the model says the L2s fetch, the recorded counter figure where one is committed, and Section 7's bound."""
    img, flt = ci.make_inputs(cfg)
    d_img = torch.from_numpy(ci.bf16_bits(img).view(np.int16).reshape(-1)).cuda()
    d_flt = torch.from_numpy(ci.bf16_bits(flt).view(np.int16).reshape(-1)).cuda()
    d_out = torch.empty(int(np.prod(cfg.out_shape)), dtype=torch.float32, device="cuda:0")
    plan = cc.cacnn_tile_plan(cfg.dims, 1)
    l2 = cc.cacnn_two_level_plan(cfg.dims, 1)
    esz = 2.0
    n_out = float(np.prod(cfg.out_shape))
    M2 = 4 * 1024 * 1024 / esz
    rep = {"workload": f"{cfg.name}: B={cfg.B} C={cfg.C} K={cfg.K} W=H={cfg.W} R=S={cfg.R} bf16",
           "chosen_a_K": l2.a_k, "chosen_walk": l2.walk, "variant": cc.cacnn_variant_name(plan.variant), "grid": plan.grid[0],
           "image_bytes": float(np.prod(cfg.image_shape)) * esz, "filter_bytes": float(np.prod(cfg.filter_shape)) * esz,
           "lp_at_M_l2": {"tile_b_c_k_w_h": [l2.lp_tile[i] for i in range(5)], "cost_words": l2.lp_cost_words,
                          "bound_words": l2.bound_words,
                          "tile_in_whole_lds_tiles_b_k_w_h": [l2.l2_tile_b, l2.l2_tile_k, l2.l2_tile_w, l2.l2_tile_h]},
           "layouts": {}}
    a, b = cc.cacnn_work_division(cfg.dims, M2, 8)
    rep["paper_division_p8_M_l2"] = {"a_B_a_K_a_W_a_H": list(a), "bound_words": b.bound}
    # four passes over the layouts, alternately forwards and backwards; per layout and pass the power-state conditioning,
    # `warmup` launches, `steps` timed ones; the figure kept is the median of the four (the clock's slow stretch between
    # a few dozen and a few hundred launches after a cold start would otherwise land on whichever layout comes first)
    cands = [(l2.cand_a_k[i], l2.cand_walk[i]) for i in range(l2.n_candidates)]
    times = {c: [] for c in cands}
    for rnd in range(4):
        for (ak, walk) in (cands if rnd % 2 == 0 else cands[::-1]):
            plan.xcd_split_k, plan.xcd_walk = ak, walk
            condition_power_state(cc, torch, ci, np, "bf16")
            for _ in range(warmup):
                cc.cacnn_conv_forward_with_plan(cfg.dims, 1, plan, d_img, d_flt, d_out)
            e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            e0.record()
            for _ in range(steps):
                cc.cacnn_conv_forward_with_plan(cfg.dims, 1, plan, d_img, d_flt, d_out)
            e1.record()
            torch.cuda.synchronize()
            times[(ak, walk)].append(e0.elapsed_time(e1) * 1e-3 / steps)
    for i, (ak, walk) in enumerate(cands):
        sec = float(np.median(times[(ak, walk)]))
        pb = cc.cacnn_parallel_bound(cfg.dims, M2, (1, ak, 1, min(8 // ak, cfg.H)))
        rep["layouts"][f"aK{ak}w{walk}"] = {
            "us": sec * 1e6, "us_min": min(times[(ak, walk)]) * 1e6, "tflops": 2.0 * cfg.macs / sec / 1e12,
            "model_bytes": esz * (l2.cand_words[i] - n_out) + 4.0 * n_out,
            "paper_parallel_bound_words_M_l2": pb.bound,
            "hbm_bytes_recorded": committed_traffic(f"{cfg.name}_aK{ak}w{walk}")}
    return rep


def pool_traffic_probe(cc, torch, ci, np, cfg):
    """As traffic_probe, for the pooling workload (max pooling): calibration copy, eviction, cold launch, warm launch."""
    n = 512 * 1024 * 1024
    src = torch.empty(n, dtype=torch.uint8, device="cuda:0").fill_(1)
    dst = torch.empty(n, dtype=torch.uint8, device="cuda:0")
    img, _ = ci.make_inputs(cfg)
    d_img = torch.from_numpy(img.reshape(-1)).cuda()
    d_out = torch.empty(int(np.prod(cfg.out_shape)), dtype=torch.float32, device="cuda:0")
    torch.cuda.synchronize()
    dst.copy_(src)
    torch.cuda.synchronize()
    evict = torch.empty(1024 * 1024 * 1024, dtype=torch.uint8, device="cuda:0").fill_(3)
    torch.cuda.synchronize()
    cc.cacnn_pool_forward(cfg.dims, 0, 1, d_img, d_out)      # cold
    torch.cuda.synchronize()
    cc.cacnn_pool_forward(cfg.dims, 0, 1, d_img, d_out)      # warm
    torch.cuda.synchronize()
    del evict
    print(json.dumps({"traffic_probe": cfg.name, "copy_bytes_each_way": n}))


def pooling_report(cc, torch, ci, np, steps, warmup, with_cpu):
    """The pooling path (Section 6 of the paper) on its workload p1, max and average: HBM-bound, so the figure is
    compulsory bytes (Image once + Out once) over time against the published HBM peak, with the oracle timed beside it.
    Five sets of buffers in rotation, 650 MB: one set alone would stay in the 256 MB last-level cache from one launch to the next."""
    cfg = ci.POOL_CONFIGS["p1"]
    img, _ = ci.make_inputs(cfg)
    d_imgs = [torch.from_numpy(img.reshape(-1)).cuda() for _ in range(5)]
    d_outs = [torch.empty(int(np.prod(cfg.out_shape)), dtype=torch.float32, device="cuda:0") for _ in d_imgs]
    d_out = d_outs[0]
    nbytes = 4 * (int(np.prod(cfg.image_shape)) + int(np.prod(cfg.out_shape)))
    rep = {"workload": f"p1: B={cfg.B} C=K={cfg.C} W=H={cfg.W} R=S={cfg.R} sigma={cfg.sigma_w} f32",
           "compulsory_bytes": nbytes, "bound": "hbm", "peak_GBps": HBM_PEAK_GBS}
    for mode, code in (("max", 1), ("avg", 0)):
        for i in range(max(warmup, 5)):
            cc.cacnn_pool_forward(cfg.dims, 0, code, d_imgs[i % 5], d_outs[i % 5])
        torch.cuda.synchronize()
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        e0.record()
        for i in range(steps):
            cc.cacnn_pool_forward(cfg.dims, 0, code, d_imgs[i % 5], d_outs[i % 5])
        e1.record()
        torch.cuda.synchronize()
        sec = e0.elapsed_time(e1) / steps * 1e-3
        rep[mode] = {"us": sec * 1e6, "GBps": nbytes / sec / 1e9, "frac_hbm_peak": nbytes / sec / 1e9 / HBM_PEAK_GBS}
    if with_cpu:
        from oracle import conv as oconv
        from oracle import pool as opool
        p = oconv.Problem(*cfg.dims)
        t0 = time.perf_counter()
        ref = opool.pool_fp64(p, img, "avg")
        dt = time.perf_counter() - t0
        got = d_out.cpu().numpy().reshape(cfg.out_shape).astype(np.float64)
        scale = opool.pool_fp64(p, np.abs(img), "avg")
        rep["cpu_baseline"] = {"value": nbytes / dt / 1e9, "unit": "GB/s", "cores": 1, "kind": "oracle",
                               "sample": f"p1 average pooling, whole workload, numpy fp64, {dt:.2f} s",
                               "max_rel_err_gpu_vs_oracle": float(np.max(np.abs(got - ref) / np.maximum(scale, 1e-300)))}
    return rep


# Mid-size and ragged layers outside the benchmark shapes' own kernels (two of the bf16 ones with 32 images are taken by the
# 32-image fixed-geometry kernels, the others by generic kernels): (dtype, B, C, K, W, H, R, S, sigma_w, sigma_h)
PLANNER_SHAPES = [
    ("bf16", 32, 1024, 256, 14, 14, 1, 1, 1, 1), ("bf16", 32, 512, 512, 7, 7, 3, 3, 1, 1), ("bf16", 32, 64, 64, 56, 56, 3, 3, 1, 1),
    ("bf16", 16, 128, 128, 28, 28, 3, 3, 1, 1), ("bf16", 40, 96, 200, 13, 11, 3, 3, 1, 1), ("bf16", 24, 48, 96, 27, 27, 5, 5, 2, 2),
    ("bf16", 128, 256, 512, 1, 1, 1, 1, 1, 1), ("bf16", 8, 256, 256, 20, 20, 3, 3, 2, 2),
    ("f32", 32, 256, 256, 14, 14, 3, 3, 1, 1), ("f32", 4, 128, 128, 28, 28, 3, 3, 1, 1), ("f32", 16, 64, 96, 30, 30, 5, 5, 1, 1),
    ("f32", 20, 40, 72, 17, 19, 3, 3, 1, 1), ("f32", 64, 16, 32, 55, 55, 7, 7, 2, 2), ("f32", 2, 64, 64, 56, 56, 3, 3, 1, 1),
    ("f32", 256, 512, 512, 1, 1, 1, 1, 1, 1), ("f32", 12, 100, 60, 25, 9, 1, 3, 1, 2),
]


# Layers the cost model's constants are fitted on (none of them is in PLANNER_SHAPES)
CALIBRATION_SHAPES = [
    ("bf16", 64, 128, 128, 14, 14, 3, 3, 1, 1), ("bf16", 16, 256, 256, 14, 14, 3, 3, 1, 1), ("bf16", 8, 64, 128, 56, 56, 1, 1, 1, 1),
    ("bf16", 32, 256, 64, 28, 28, 1, 1, 1, 1), ("bf16", 128, 64, 64, 7, 7, 3, 3, 1, 1), ("bf16", 4, 512, 512, 14, 14, 3, 3, 1, 1),
    ("bf16", 48, 80, 160, 12, 10, 3, 3, 1, 1), ("bf16", 16, 32, 64, 30, 30, 5, 5, 1, 1), ("bf16", 32, 96, 96, 16, 16, 3, 3, 2, 2),
    ("bf16", 64, 512, 128, 4, 4, 3, 3, 1, 1), ("bf16", 256, 128, 256, 1, 1, 1, 1, 1, 1), ("bf16", 20, 200, 72, 9, 13, 3, 1, 1, 1),
    ("bf16", 8, 128, 128, 24, 24, 3, 3, 1, 1), ("bf16", 32, 32, 32, 56, 56, 3, 3, 1, 1), ("bf16", 16, 64, 256, 20, 20, 1, 1, 1, 1),
    ("bf16", 96, 48, 48, 10, 10, 5, 5, 2, 2),
    ("f32", 16, 128, 128, 14, 14, 3, 3, 1, 1), ("f32", 8, 64, 64, 28, 28, 3, 3, 1, 1), ("f32", 32, 32, 64, 20, 20, 5, 5, 1, 1),
    ("f32", 1, 64, 64, 56, 56, 3, 3, 1, 1), ("f32", 64, 256, 128, 4, 4, 1, 1, 1, 1), ("f32", 8, 24, 48, 33, 31, 3, 3, 2, 2),
    ("f32", 4, 96, 96, 24, 24, 3, 3, 1, 1), ("f32", 128, 128, 256, 1, 1, 1, 1, 1, 1), ("f32", 10, 50, 70, 15, 11, 3, 5, 1, 2),
    ("f32", 32, 8, 32, 48, 48, 7, 7, 2, 2), ("f32", 16, 192, 64, 12, 12, 1, 1, 1, 1), ("f32", 2, 128, 128, 28, 28, 3, 3, 1, 1),
]


def planner_sweep(cc, torch, ci, np, shapes):
    """Every kernel variant that accepts each shape, with the contraction tile the cost model likes best for it: the
    model's estimate next to the measured launch time.  The data the model's constants are fitted to and judged by."""
    print("sweep | dtype B C K W H R S sw sh | variant | b_c b_r b_s | model us | measured us | model terms: tiles per CU, "
          "MFMA, staging, slices, Out drain (CU cycles)")
    rows = {}
    for sh in shapes:
        dtype, dims = sh[0], sh[1:]
        cfg = ci.custom("sweep", *dims, dtype=dtype, dist="normal", seed=4)
        _, _, d_img, d_flt, d_out = upload_config(torch, ci, np, cfg)
        dt = 0 if dtype == "f32" else 1
        for vi in range(cc.cacnn_variant_count()):
            try:
                plan, model_us, terms = cc.cacnn_plan_variant(dims, dt, vi, True)
                for _ in range(3):
                    cc.cacnn_conv_forward_with_plan(dims, dt, plan, d_img, d_flt, d_out)
            except cc.CacnnError:
                continue
            e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            e0.record()
            for _ in range(12):
                cc.cacnn_conv_forward_with_plan(dims, dt, plan, d_img, d_flt, d_out)
            e1.record()
            torch.cuda.synchronize()
            print(f"sweep | {dtype} {' '.join(str(v) for v in dims)} | {cc.cacnn_variant_name(vi)} | {plan.b_c} {plan.b_r} "
                  f"{plan.b_s} | {model_us:.2f} | {e0.elapsed_time(e1) * 1e3 / 12:.2f} | "
                  f"{' '.join(f'{t:.6g}' for t in terms)}", flush=True)
            tag = cc.cacnn_variant_name(vi).split()[1]
            if not tag.startswith("fx"):
                family = f"{dtype} {'one-tile' if tag.startswith('k') else tag}"
                per_cu, t_mfma, t_stage, n_ct, t_out = terms
                rows.setdefault(family, []).append(
                    ([per_cu * t_mfma, per_cu * t_stage, per_cu * n_ct, t_out / max(1.0, min(per_cu, 4.0)), 1.0],
                     e0.elapsed_time(e1) * 1e3 / 12 * 2400.0))
    # the fit the cost model's coefficients come from: per kernel family, non-negative least squares on the relative error
    from scipy.optimize import nnls
    print("fit | family | cycles per MFMA cycle, per staging cycle, per slice, per Out-drain cycle, constant | rms log error | rows")
    for family in sorted(rows):
        A = np.array([[f / meas for f in feats] for feats, meas in rows[family]])
        x, _ = nnls(A, np.ones(len(A)))
        err = np.log(np.maximum(A @ x, 1e-9))
        print(f"fit | {family} | {' '.join(f'{c:.4g}' for c in x)} | {float(np.sqrt(np.mean(err ** 2))):.3f} | {len(A)}")


# layers that the fixed-geometry kernels added for 1 x 1 filters, for 32-image tiles and for tiles that overhang Out take
# (beside the benchmark shapes' own)
ONE_BY_ONE_SHAPES = [
    ("f32", 8, 256, 256, 14, 14, 1, 1, 1, 1), ("f32", 32, 512, 128, 28, 28, 1, 1, 1, 1), ("f32", 16, 64, 256, 56, 56, 1, 1, 1, 1),
    ("f32", 64, 1024, 256, 14, 14, 1, 1, 1, 1),
    ("bf16", 64, 1024, 256, 14, 14, 1, 1, 1, 1), ("bf16", 128, 256, 512, 7, 7, 1, 1, 1, 1), ("bf16", 64, 512, 2048, 7, 7, 1, 1, 1, 1),
    ("bf16", 64, 64, 256, 56, 56, 1, 1, 1, 1), ("bf16", 256, 2048, 512, 7, 7, 1, 1, 1, 1),
    # 32 images (or a multiple that is not one of 64): the fixed-geometry bf16 kernels with 32-image tiles take these
    ("bf16", 32, 128, 128, 56, 56, 3, 3, 1, 1), ("bf16", 32, 512, 512, 14, 14, 3, 3, 1, 1), ("bf16", 96, 128, 128, 28, 28, 3, 3, 1, 1),
    ("bf16", 32, 256, 256, 28, 28, 3, 3, 1, 1), ("bf16", 32, 256, 1024, 14, 14, 1, 1, 1, 1),
    # W, H, K (or B) that no tile divides: the bf16 kernels that load the Image straight into LDS mask their Out stores
    ("bf16", 128, 256, 384, 13, 13, 3, 3, 1, 1), ("bf16", 128, 384, 256, 13, 13, 3, 3, 1, 1), ("bf16", 64, 96, 256, 27, 27, 1, 1, 1, 1),
    ("bf16", 64, 2048, 1000, 1, 1, 1, 1, 1, 1), ("bf16", 64, 64, 192, 55, 55, 3, 3, 1, 1), ("bf16", 64, 128, 160, 17, 17, 3, 3, 1, 1),
    ("bf16", 128, 512, 512, 13, 13, 1, 1, 1, 1), ("bf16", 64, 160, 320, 10, 10, 3, 3, 1, 1),
    # fewer images than a tile, or a count that no tile divides (multiples of 8)
    ("bf16", 48, 64, 64, 14, 14, 3, 3, 1, 1), ("bf16", 8, 512, 512, 7, 7, 3, 3, 1, 1),
    ("bf16", 24, 64, 64, 56, 56, 3, 3, 1, 1), ("bf16", 16, 256, 512, 14, 14, 1, 1, 1, 1),
    # 1 x 1 filters with strides
    ("bf16", 64, 256, 512, 14, 14, 1, 1, 2, 2), ("bf16", 32, 512, 1024, 7, 7, 1, 1, 2, 2), ("bf16", 128, 64, 128, 28, 28, 1, 1, 2, 2),
    # 3 x 3 filters with strides 2
    ("bf16", 64, 128, 128, 28, 28, 3, 3, 2, 2), ("bf16", 64, 256, 256, 14, 14, 3, 3, 2, 2), ("bf16", 128, 512, 512, 7, 7, 3, 3, 2, 2),
    # C a multiple of 8 but not of 32 (the first four: 16 mod 32)
    ("bf16", 128, 80, 192, 28, 28, 3, 3, 1, 1), ("bf16", 64, 144, 288, 14, 14, 1, 1, 1, 1), ("bf16", 64, 48, 128, 56, 56, 3, 3, 1, 1),
    ("bf16", 64, 16, 64, 112, 112, 3, 3, 1, 1), ("bf16", 64, 40, 120, 28, 28, 1, 1, 1, 1), ("bf16", 64, 120, 40, 28, 28, 1, 1, 1, 1),
    ("bf16", 64, 24, 72, 56, 56, 3, 3, 1, 1), ("bf16", 128, 72, 72, 28, 28, 3, 3, 1, 1),
    # the same for the fp32 kernel with 16 x 16 blocks
    ("f32", 16, 256, 384, 13, 13, 3, 3, 1, 1), ("f32", 8, 96, 256, 27, 27, 1, 1, 1, 1), ("f32", 32, 128, 160, 17, 17, 3, 3, 1, 1),
    ("f32", 8, 2048, 1000, 1, 1, 1, 1, 1, 1), ("f32", 8, 256, 512, 14, 14, 1, 1, 2, 2), ("f32", 16, 64, 128, 28, 28, 1, 1, 2, 2),
    # other filters, which the kernels compiled for 1 x 1 filters take one tap at a time: 5 x 5, 1 x 7 and 7 x 1, 7 x 7,
    # 5 x 5 with strides 2, C = 16 mod 32; fp32 3 x 3 with strides 2 and 5 x 5
    ("bf16", 64, 96, 256, 27, 27, 5, 5, 1, 1), ("bf16", 32, 128, 128, 17, 17, 1, 7, 1, 1), ("bf16", 32, 128, 128, 17, 17, 7, 1, 1, 1),
    ("bf16", 64, 64, 64, 28, 28, 7, 7, 1, 1), ("bf16", 64, 64, 128, 14, 14, 5, 5, 2, 2), ("bf16", 64, 48, 128, 27, 27, 5, 5, 1, 1),
    ("f32", 16, 64, 128, 14, 14, 3, 3, 2, 2), ("f32", 16, 96, 256, 27, 27, 5, 5, 1, 1),
    # stem layers (7 x 7, strides 2, three channels) that the stem kernel's tile of 32 images x 2 x 2 positions x 64 channels
    # does not divide
    ("f32", 16, 3, 64, 112, 112, 7, 7, 2, 2), ("f32", 64, 3, 96, 109, 109, 7, 7, 2, 2),
    # fewer images than a tile together with a K that no tile divides, odd batch sizes (the planner's worst rows are here:
    # shallow 56 x 56 layers with 40 or 24 images, which are bound by their Out stores and run best on 8-image tiles)
    ("bf16", 40, 96, 192, 56, 56, 1, 1, 1, 1), ("bf16", 24, 40, 192, 56, 56, 1, 1, 1, 1), ("bf16", 8, 512, 256, 20, 20, 5, 5, 2, 2),
    ("bf16", 32, 72, 72, 28, 28, 5, 5, 1, 1), ("bf16", 16, 192, 136, 14, 14, 5, 5, 1, 1), ("bf16", 24, 512, 136, 28, 28, 3, 3, 2, 2),
    ("bf16", 40, 512, 192, 28, 28, 3, 3, 1, 1), ("bf16", 8, 64, 136, 28, 28, 3, 3, 2, 2),
    # fp32 with C a multiple of 4 but not of 16
    ("f32", 16, 24, 96, 56, 56, 3, 3, 1, 1), ("f32", 8, 40, 120, 28, 28, 1, 1, 1, 1), ("f32", 16, 72, 72, 28, 28, 3, 3, 1, 1),
]


def padded_shapes():
    """36 seeded random bf16 layers on which a 64- or 32-image tile is partly empty: 8 to 40 images, output-channel
    counts that no k-tile divides among them, 1 x 1 to 1 x 7 filters, strides 1 and 2."""
    import random
    rng = random.Random(5)
    shapes = []
    while len(shapes) < 36:
        B = rng.choice([8, 16, 24, 32, 40])
        C = rng.choice([32, 40, 64, 72, 96, 128, 192, 256, 512])
        K = rng.choice([40, 64, 72, 96, 136, 192, 256, 512])
        W = rng.choice([7, 14, 20, 28, 56])
        R, S = rng.choice([(1, 1), (3, 3), (3, 3), (5, 5), (1, 7)])
        st = rng.choice([1, 1, 2])
        if 3e8 < B * C * K * W * W * R * S < 4e10:
            shapes.append(("bf16", B, C, K, W, W, R, S, st, st))
    return shapes


def planner_compare(cc, torch, ci, np, padded=False):
    """The planner's pick against the fastest of all kernel variants (cacnn_tune) on PLANNER_SHAPES; the planner is the
    one the environment selects (CACNN_PLANNER unset: the calibrated cycle model; lp: the tile sized from the Section 5
    LP at the gfx950 budget).  One row per shape, then the geometric mean of the ratios.  On ONE_BY_ONE_SHAPES, which the
    fixed-geometry kernels take, the row also has the fastest of the generic variants.  padded: on padded_shapes()
    instead, the summary over all of them."""
    mode = os.environ.get("CACNN_PLANNER", "model")

    def timed(fn, n=60, w=10):
        for _ in range(w):
            fn()
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        e0.record()
        for _ in range(n):
            fn()
        e1.record()
        torch.cuda.synchronize()
        return e0.elapsed_time(e1) / n * 1e3

    ratios = []
    print("mode | dtype B C K W H R S sw sh | planner's variant [b_c b_r b_s] us | fastest variant [b_c b_r b_s] us | ratio")
    for sh in (padded_shapes() if padded else PLANNER_SHAPES + ONE_BY_ONE_SHAPES):
        dtype, dims = sh[0], sh[1:]
        cfg = ci.custom("cmp", *dims, dtype=dtype, dist="normal", seed=3)
        _, _, d_img, d_flt, d_out = upload_config(torch, ci, np, cfg)
        dt = 0 if dtype == "f32" else 1
        plan = cc.cacnn_tile_plan(dims, dt)
        tuned = cc.cacnn_tune(dims, dt, d_img, d_flt, d_out)
        # the two timed in turns, twice: the clock the chip settles at depends on what ran just before (the sweep inside
        # cacnn_tune leaves it higher than the upload does), which would otherwise favour whichever comes second
        t_plan = t_tune = 0.0
        for _ in range(2):
            t_plan += 0.5 * timed(lambda: cc.cacnn_conv_forward_with_plan(dims, dt, plan, d_img, d_flt, d_out), n=30)
            t_tune += 0.5 * timed(lambda: cc.cacnn_conv_forward_with_plan(dims, dt, tuned, d_img, d_flt, d_out), n=30)
        generic = ""
        if padded:
            ratios.append(t_plan / t_tune)
        if sh in PLANNER_SHAPES:
            ratios.append(t_plan / t_tune)                # the summary line is about the generic kernels' cost model
        else:
            # what the fixed-geometry kernel is worth on this layer: the fastest of the other variants
            best = None
            for vi in range(cc.cacnn_variant_count()):
                if " fx" in cc.cacnn_variant_name(vi):
                    continue
                try:
                    gplan, _ = cc.cacnn_plan_variant(dims, dt, vi)
                    t = timed(lambda: cc.cacnn_conv_forward_with_plan(dims, dt, gplan, d_img, d_flt, d_out), n=20, w=3)
                except cc.CacnnError:
                    continue
                if best is None or t < best[0]:
                    best = (t, vi)
            if best is not None:
                generic = f" | fastest generic variant: {cc.cacnn_variant_name(best[1])} {best[0]:.2f} ({best[0] / t_plan:.2f} x the planner's)"
        print(f"{mode} | {dtype} {' '.join(str(v) for v in dims)} | {cc.cacnn_variant_name(plan.variant)} "
              f"[{plan.b_c}, {plan.b_r}, {plan.b_s}] {t_plan:.2f} | {cc.cacnn_variant_name(tuned.variant)} "
              f"[{tuned.b_c}, {tuned.b_r}, {tuned.b_s}] {t_tune:.2f} | {t_plan / t_tune:.3f}{generic}", flush=True)
    gm = float(np.exp(np.mean(np.log(ratios))))
    print(f"{mode}: geometric mean of the ratios {gm:.3f}, worst {max(ratios):.2f}, within 15 % of the fastest on "
          f"{sum(1 for r in ratios if r <= 1.15)} of {len(ratios)}")


def main():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=500, help="timed launches")
    ap.add_argument("--warmup", type=int, default=50, help="untimed launches in front of the timed ones")
    ap.add_argument("--no-conditioning", action="store_true",
                    help="skip the 0.3 s of register-only MFMA load that precedes each shape's warm-up launches (a cold "
                         "board's power management makes the first hundreds of launches slower)")
    ap.add_argument("--workload", default="c5", choices=["c1", "c2", "c3", "c4", "c5", "p1", "d1", "d2"],
                    help="c1..c5: the convolution shapes (c5, the largest, is the headline); p1: the pooling workload; "
                         "d1, d2: the two-level workloads (a Filter-heavy layer on 64 and 256 images, every layout of an "
                         "XCD's run of tiles)")
    ap.add_argument("--xcd-split-k", type=int, default=0,
                    help="with --traffic-probe: force this division of the XCDs over the output channels (0: planner's)")
    ap.add_argument("--xcd-walk", type=int, default=0,
                    help="with --traffic-probe and --xcd-split-k: order inside an XCD's run (0: k-tiles fastest, 1: positions)")
    ap.add_argument("--no-shapes", action="store_true", help="time only the headline workload")
    ap.add_argument("--no-cpu", action="store_true", help="skip the cpu_baseline leg")
    ap.add_argument("--traffic-probe", action="store_true",
                    help="for rocprofv3 --pmc runs: one 512 MiB device copy (calibration), a cache-evicting 1 GiB fill, "
                         "then one cold and one warm launch of the workload; prints nothing but a marker line")
    ap.add_argument("--two-level", action="store_true",
                    help="with --workload c4 or c5: time every layout of an XCD's run of tiles that the two-level plan prices "
                         "(what --workload d1 / d2 always do)")
    ap.add_argument("--planner-sweep", choices=["calibration", "test"], default=None,
                    help="time every kernel variant on the calibration layers (or on the --planner-compare layers) and print "
                         "the cost model's estimate next to each; no JSON line")
    ap.add_argument("--planner-compare-padded", action="store_true",
                    help="the same comparison on 36 seeded random bf16 layers with 8 to 40 images and output-channel counts "
                         "that no tile divides; no JSON line")
    ap.add_argument("--planner-compare", action="store_true",
                    help="time the planner's pick against cacnn_tune's on sixteen mid-size and ragged layers and print a "
                         "table (the planner is the one CACNN_PLANNER selects); no JSON line")
    args = ap.parse_args()
    if args.gpus != 1:
        print("bench.py: this build runs on one GPU only (the path shards over b or k with no exchange step, "
              "but no multi-GPU run is part of it); use --gpus 1", file=sys.stderr)
        sys.exit(2)

    import numpy as np
    import torch

    import cacnn_inputs as ci
    import paper_1802_06905_amd as cc      # raises if libcacnn.so is not built: no fallback

    if not torch.cuda.is_available():
        print("bench.py: no GPU visible", file=sys.stderr)
        sys.exit(2)
    torch.cuda.set_device(0)

    if args.planner_sweep:
        planner_sweep(cc, torch, ci, np, {"calibration": CALIBRATION_SHAPES, "test": PLANNER_SHAPES}[args.planner_sweep])
        return
    if args.planner_compare or args.planner_compare_padded:
        planner_compare(cc, torch, ci, np, padded=args.planner_compare_padded)
        return
    if args.workload == "p1":
        pcfg = ci.POOL_CONFIGS["p1"]
        if args.traffic_probe:
            pool_traffic_probe(cc, torch, ci, np, pcfg)
            return
        rep = pooling_report(cc, torch, ci, np, args.steps, args.warmup, not args.no_cpu)
        out = {"metric": "max-pooling GB/s at 1 MI355X (compulsory bytes / time)", "value": rep["max"]["GBps"],
               "unit": "GB/s", "n_gpus": 1, "steps": args.steps, "warmup": args.warmup,
               "ms_per_step": rep["max"]["us"] * 1e-3, "higher_is_better": True, "scaling": "weak", "vs_baseline": None,
               "dtype": "f32", "data": "synthetic", "config": {"workload": rep["workload"]},
               "roofline": {"bound": "hbm", "achieved": rep["max"]["GBps"], "peak": HBM_PEAK_GBS, "unit": "GB/s",
                            "frac": rep["max"]["frac_hbm_peak"], "traffic": committed_traffic("p1")},
               "average_pooling": rep["avg"]}
        if "cpu_baseline" in rep:
            out["cpu_baseline"] = rep["cpu_baseline"]
        print(json.dumps(out))
        return
    if args.workload in ("d1", "d2") or (args.two_level and args.workload in ("c4", "c5") and not args.traffic_probe):
        dcfg = ci.DIVISION_CONFIGS[args.workload] if args.workload in ci.DIVISION_CONFIGS else ci.CONFIGS[args.workload]
        if args.traffic_probe:
            traffic_probe(cc, torch, ci, np, dcfg, args.xcd_split_k, args.xcd_walk)
            return
        rep = division_report(cc, torch, ci, np, dcfg, args.steps, args.warmup)
        best = rep["layouts"][f"aK{rep['chosen_a_K']}w{rep['chosen_walk']}"]
        print(json.dumps({"metric": "conv TFLOP/s at 1 MI355X", "value": best["tflops"], "unit": "TFLOP/s", "n_gpus": 1,
                          "steps": args.steps, "warmup": args.warmup, "ms_per_step": best["us"] * 1e-3,
                          "higher_is_better": True, "scaling": "weak", "vs_baseline": None, "dtype": "bf16",
                          "data": "synthetic", "config": {"workload": rep["workload"], "variant": rep["variant"]},
                          "roofline": {"bound": "mfma", "achieved": best["tflops"], "peak": MFMA_PEAK_TFLOPS["bf16"],
                                       "unit": "TFLOP/s", "frac": best["tflops"] / MFMA_PEAK_TFLOPS["bf16"],
                                       "traffic": best["hbm_bytes_recorded"]},
                          "two_level": rep}))
        return
    cfg = ci.CONFIGS[args.workload]
    if args.traffic_probe:
        traffic_probe(cc, torch, ci, np, cfg, args.xcd_split_k, args.xcd_walk)
        return
    # inputs first (host work), so that nothing idles the GPU between conditioning, warm-up and the timed launches
    names = [cfg.name] if args.no_shapes else list(ci.CONFIGS)
    buffers = {n: upload_config(torch, ci, np, ci.CONFIGS[n]) for n in names}
    torch.cuda.synchronize()
    # (with --no-conditioning the sustained-rate loops run after the timed launches instead: they are a matrix load too)
    sustained = None if args.no_conditioning else machine_sustained(cc, torch, ci, np)
    sec, wall = time_config(cc, torch, ci, np, cfg, args.steps, args.warmup, buffers[cfg.name],
                            condition=not args.no_conditioning)
    if sustained is None:
        sustained = machine_sustained(cc, torch, ci, np)
    img, flt, _, _, d_out = buffers[cfg.name]
    head = shape_report(cc, cfg, sec)
    head["frac_mfma_sustained"] = head["tflops"] / sustained[f"mfma_{cfg.dtype}_tflops"]
    add_unit_mix(head, cfg, sustained)

    # parity of the timed launch against the oracle (also the cpu_baseline leg)
    result = {
        "metric": "conv TFLOP/s at 1 MI355X", "value": head["tflops"], "unit": "TFLOP/s", "n_gpus": 1,
        "steps": args.steps, "warmup": args.warmup, "ms_per_step": sec * 1e3, "higher_is_better": True,
        "scaling": "weak", "vs_baseline": None, "dtype": cfg.dtype if cfg.dtype == "f32" else "bf16",
        "data": "synthetic",
        "config": {"workload": f"{cfg.name}: B={cfg.B} C={cfg.C} K={cfg.K} W=H={cfg.W} R=S={cfg.R} "
                               f"sigma={cfg.sigma_w} {cfg.dtype} in, fp32 accumulate/out",
                   "variant": head["variant"], "grid": head["grid"], "lds_bytes": head["lds_bytes"]},
        "roofline": {"bound": "mfma", "achieved": head["tflops"], "peak": MFMA_PEAK_TFLOPS[cfg.dtype],
                     "unit": "TFLOP/s", "frac": head["frac_mfma_peak"], "traffic": head["hbm_bytes_recorded"],
                     "wall_us_per_step": wall * 1e6, "frac_of_sustained_mfma": head["frac_mfma_sustained"]},
        "machine_sustained": sustained,
    }
    if not args.no_cpu:
        base, ref, ab, k_use = cpu_baseline(cfg, img, flt, np)
        got = d_out.cpu().numpy().reshape(cfg.out_shape)[:k_use].astype(np.float64)
        err = float(np.max(np.abs(got - ref) / np.maximum(ab, 1e-300)))
        base["max_rel_err_gpu_vs_oracle"] = err
        result["cpu_baseline"] = base
    if not args.no_shapes:
        shapes = {}
        for name, c in ci.CONFIGS.items():
            if name == cfg.name:
                shapes[name] = head
                continue
            s, _ = time_config(cc, torch, ci, np, c, args.steps, args.warmup, buffers[name],
                               condition=not args.no_conditioning)
            shapes[name] = shape_report(cc, c, s)
            shapes[name]["frac_mfma_sustained"] = shapes[name]["tflops"] / sustained[f"mfma_{c.dtype}_tflops"]
            add_unit_mix(shapes[name], c, sustained)
            shapes[name]["other_fixed_geometry_variants_us"] = alternative_variants_us(
                cc, torch, c, buffers[name], args.steps, args.warmup)
            if name == "c1":
                shapes[name]["us_per_launch_in_a_hip_graph"] = graph_replay_us(cc, torch, ci, np, c, buffers[name])
        # (the headline shape's extras last, so that its own timed region and parity check come first)
        condition_power_state(cc, torch, ci, np, cfg.dtype)
        head["us_per_launch_in_a_hip_graph"] = graph_replay_us(cc, torch, ci, np, cfg, buffers[cfg.name], launches=100, replays=5)
        head["other_fixed_geometry_variants_us"] = alternative_variants_us(cc, torch, cfg, buffers[cfg.name],
                                                                           args.steps, args.warmup)
        result["shapes"] = shapes
        result["pooling"] = pooling_report(cc, torch, ci, np, args.steps, args.warmup, not args.no_cpu)
    print(json.dumps(result))


if __name__ == "__main__":
    main()
