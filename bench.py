#!/usr/bin/env python3
"""Benchmark of the tensorized-approximation (TA) long-range TEI hot path on
one MI355X.

One step = one pass of the hot path over the Nb = 400 workload (40 atoms with
s, p, d shells, 80200 pairs, omega = 0.3, nq = 32, n = 40, L = 16): FP64
quadrature tables and moments, operand preparation, and the fused assembly of
the full 80200 x 80200 B, in the headline arithmetic (split FP16, 3 products).
`value` = stored B entries per second of that step, inputs resident on the
device.  The same line reports the FP64 / FP32 / BF16 forms of the same step,
FP64 and FP32 with a degree per quadrature node (the paper's N_i, each
factor within 1e-8 on the box), the step and the J-build over the pairs that
screening keeps (prefactor above 1e-12), the orbital-basis Coulomb matrix
of 16 orbitals at Nb = 1000, the batched persistent assembly of 64 molecules (graph replay vs one launch
sequence per molecule), the J-build through the grid tensor (Nb = 1000), the
error of every form against the FP64 oracle on sampled entries, the roofline
of the dominant kernel, and the oracle timed on the host cores.

    python bench.py [--gpus 1] [--steps K] [--warmup W] [--only-headline] [--no-cpu]
"""
import argparse
import dataclasses
import hashlib
import json
import os
import sys
import time

ROOT = os.path.dirname(os.path.abspath(__file__))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)

METRIC = "long-range TEI entries/s: split-BF16/FP32 vs FP64 GPU, at stated rel. error"
# MI355X published dense peaks, TFLOP/s
PEAK_TFLOPS = {"fp64": 78.6, "fp32": 157.3, "bf16x3": 2500.0, "bf16x6": 2500.0, "f16x3": 2500.0}
HBM_PEAK_GBS = 8000.0
# tolerance of the per-node degree leg: each node's factor moves by at most
# this much on the box (below the degree-40 interpolation error at omega 0.3)
DEGREE_TOL = 1e-8
# tolerance of the low-rank compression legs: directions of the stacked
# moments with sigma_r <= this * sigma_1 are dropped
RANK_TOL = 1e-7
# the J-build legs cut at a looser tolerance: the grid kernels work in tiles
# of 16 directions, so the compression pays there once R <= 32 of n = 48
RANK_TOL_J = 1e-5
# screening threshold of the screened legs: pairs whose Gaussian product
# prefactor is at most this are dropped
SCREEN_TAU = 1e-12
# orbitals of the orbital-basis Coulomb matrix leg
NORB = 16
# adaptive integration boxes: support cut and number of boxes (the paper's
# figure of the support distribution uses 1e-20)
PARTS_TAU = 1e-20
PARTS_N = 4


def log(msg):
    print(f"[bench] {msg}", file=sys.stderr, flush=True)


def algorithmic_flops(npair, nq, n):
    """Unique entries x nodes x (three length-n dot products + two Hadamard
    products + the weighted accumulation) = npair(npair+1)/2 * nq * (6n + 4)."""
    return npair * (npair + 1) / 2 * nq * (6 * n + 4)


def algorithmic_flops_degrees(npair, nk):
    """As algorithmic_flops with node k contracting N_k indices:
    npair(npair+1)/2 * sum_k (6 N_k + 4)."""
    return npair * (npair + 1) / 2 * float(sum(6 * int(x) + 4 for x in nk))


def traffic_from_profiles(kernel_src_sha, workload):
    """HBM bytes per launch from committed counter summaries, or None when
    the kernel source changed since they were taken."""
    path = os.path.join(ROOT, "profiles", "traffic.json")
    if not os.path.exists(path):
        return None
    try:
        data = json.load(open(path))
    except Exception:
        return None
    rec = data.get(workload)
    if not rec or rec.get("kernel_src_sha") != kernel_src_sha:
        return None
    return rec.get("bytes_per_launch")


def src_sha():
    """Hash of what the dominant kernel is built from: its source, the shared
    header and the build flags."""
    h = hashlib.sha256()
    for f in ("csrc/k_assemble16.hip", "csrc/tai_internal.h", "build.py"):
        h.update(open(os.path.join(ROOT, "paper_2210_13069_amd", f), "rb").read())
    return h.hexdigest()[:16]


def load_j_fixture(name="jbuild1000_J.json"):
    """(pairs [m][2], J [m]) of the Nb = 1000 J workload from the oracle's
    stored entries, or None if the file is absent."""
    import numpy as np
    path = os.path.join(ROOT, "tests", "golden", name)
    if not os.path.exists(path):
        return None
    g = json.load(open(path))
    return np.asarray(g["pairs"], dtype=np.int64), np.asarray(g["J"], dtype=np.float64)


def stage_ms(stages, steps):
    """HIP-event time of each library stage per step (a stage may be timed in
    several sections per call)."""
    return {k: round(v[0] / max(1, steps), 4) for k, v in stages.items()}


def main():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=5)
    ap.add_argument("--warmup", type=int, default=2)
    ap.add_argument("--prec", default="f16x3", help="headline arithmetic")
    ap.add_argument("--only-headline", action="store_true", help="skip the comparison paths")
    ap.add_argument("--no-cpu", action="store_true", help="skip the oracle CPU baseline")
    ap.add_argument("--cpu-seconds", type=float, default=20.0, help="target length of the oracle sample")
    ap.add_argument("--calibrate-copy", type=int, default=0, metavar="MIB",
                    help="only run a plain device copy of MIB mebibytes (counter calibration)")
    args = ap.parse_args()
    world = int(os.environ.get("WORLD_SIZE", "1"))
    if args.gpus != 1 or world != 1:
        print("bench.py: runs on one GPU only (across GPUs the assembly tiles and the J pairs would be "
              "sharded, with one all-reduce of the n^3 grid density for J). Use --gpus 1.",
              file=sys.stderr)
        sys.exit(2)

    import numpy as np
    import torch

    from paper_2210_13069_amd import inputs as I
    from paper_2210_13069_amd import tai

    assert torch.cuda.is_available(), "bench.py needs a GPU"
    torch.cuda.set_device(0)
    dev = torch.device("cuda", 0)
    if args.calibrate_copy:
        nbytes = args.calibrate_copy << 20
        src = torch.ones(nbytes // 4, dtype=torch.float32, device=dev)
        dst = torch.empty_like(src)
        torch.cuda.synchronize()
        dst.copy_(src)
        torch.cuda.synchronize()
        print(json.dumps({"copy_bytes_read": nbytes, "copy_bytes_written": nbytes}), flush=True)
        return
    ctx = tai.Context(0)
    K, W = args.steps, args.warmup
    head = tai.PREC_BY_NAME[args.prec]

    # ---------------- headline workload --------------------------------------
    b, P = I.spd400(omega=0.3)
    npair, n, nq = b.npair, P.n, P.nq
    ba = tai.BasisArrays(b)
    M = torch.empty((3, n, npair), dtype=torch.float64, device=dev)
    # B rows start on 64-byte boundaries (row stride rounded up to 16 entries)
    ldb = tai.aligned_ldb(npair)
    B32 = torch.empty((npair, ldb), dtype=torch.float32, device=dev)
    rng = np.random.default_rng(11)
    sp = np.concatenate([rng.integers(0, npair, 240), [0, npair - 1]])
    sq = np.concatenate([rng.integers(0, npair, 240), [npair - 1, 0]])
    spt = torch.as_tensor(sp, device=dev)
    sqt = torch.as_tensor(sq, device=dev)

    def run_steps(prec, Bbuf, steps, warmup, Pw=P):
        params = tai.make_params(Pw, prec)
        for _ in range(warmup):
            ctx.moments(ba, Pw, M)
            ctx.assemble_B(M, npair, params, Bbuf, ldb)
        torch.cuda.synchronize()
        ctx.profile_enable(True)
        t0 = time.perf_counter()
        for _ in range(steps):
            ctx.moments(ba, Pw, M)
            ctx.assemble_B(M, npair, params, Bbuf, ldb)
        torch.cuda.synchronize()
        t1 = time.perf_counter()
        stages = {s: ctx.profile_read(s) for s in ("nodes", "moments", "compress", "pack", "project", "assemble")}
        ctx.profile_enable(False)
        ms = (t1 - t0) * 1e3 / steps
        sample = Bbuf[spt, sqt].double().cpu().numpy()
        return ms, stages, sample

    log(f"headline {args.prec}: Nb={b.nb} npair={npair} steps={K} warmup={W}")
    Bhead = B32 if head != tai.FP64 else torch.empty((npair, ldb), dtype=torch.float64, device=dev)
    ms_head, st_head, samp_head = run_steps(head, Bhead, K, W)
    if head == tai.FP64:
        del Bhead
    asm_ms = st_head["assemble"][0] / max(1, st_head["assemble"][1])
    entries = float(npair) * npair
    value = entries / (ms_head / 1e3)
    log(f"headline {ms_head:.2f} ms/step, assemble kernel {asm_ms:.2f} ms")

    flops = algorithmic_flops(npair, nq, n)
    achieved = flops / (asm_ms / 1e3) / 1e12
    peak = PEAK_TFLOPS[args.prec]
    roofline = {"bound": "mfma", "achieved": round(achieved, 3), "peak": peak, "unit": "TFLOP/s",
                "frac": round(achieved / peak, 5), "traffic": traffic_from_profiles(src_sha(), "spd400"),
                "kernel": "assemble16_kernel" if args.prec in ("f16x3", "bf16x3", "bf16x6") else "assemble_kernel",
                "flops_per_launch": flops,
                "launch_ms": round(asm_ms, 4)}

    paths = {args.prec: {"ms_per_step": round(ms_head, 3), "entries_per_s": value,
                         "stage_ms": stage_ms(st_head, K)}}
    samples = {args.prec: samp_head}
    samples_w1 = {}
    degrees = None
    compressed = None
    omega1 = None

    if not args.only_headline:
        B64 = torch.empty((npair, ldb), dtype=torch.float64, device=dev)
        for name in ("fp64", "fp32", "bf16x6", "bf16x3"):
            if name == args.prec:
                continue
            prec = tai.PREC_BY_NAME[name]
            steps = max(1, K // 2)
            log(f"path {name}: steps={steps}")
            ms, st, samp = run_steps(prec, B64 if prec == tai.FP64 else B32, steps, 1)
            paths[name] = {"ms_per_step": round(ms, 3), "entries_per_s": entries / (ms / 1e3),
                           "stage_ms": stage_ms(st, steps)}
            samples[name] = samp
        # per-node degrees N_k (the paper's N_i): FP64 and FP32 contract only
        # each node's leading coefficient indices
        Pd = dataclasses.replace(P, degree_tol=DEGREE_TOL)
        nk = tai.degrees(Pd)[0].cpu().numpy()
        deg_flops = algorithmic_flops_degrees(npair, nk)
        degrees = {"degree_tol": DEGREE_TOL, "N_k": nk.tolist(), "flops_per_launch": deg_flops}
        for name in ("fp64", "fp32"):
            prec = tai.PREC_BY_NAME[name]
            steps = max(1, K // 2)
            log(f"per-node degrees {name}: steps={steps}")
            ms, st, samp = run_steps(prec, B64 if prec == tai.FP64 else B32, steps, 1, Pd)
            a_ms = st["assemble"][0] / max(1, st["assemble"][1])
            degrees[name] = {"ms_per_step": round(ms, 3), "entries_per_s": entries / (ms / 1e3),
                             "stage_ms": stage_ms(st, steps),
                             "assemble_tflops_algorithmic": round(deg_flops / (a_ms / 1e3) / 1e12, 2)}
            samples[name + "_degrees"] = samp
        # low-rank compression of the moments (section 6.1): every path
        # contracts R < n directions of one SVD basis
        Pc = dataclasses.replace(P, rank_tol=RANK_TOL)
        ctx.moments(ba, P, M)
        rank = ctx.compress(M, npair, Pc)
        cmp_flops = algorithmic_flops(npair, nq, rank)
        compressed = {"rank_tol": RANK_TOL, "rank": rank, "n": n, "flops_per_launch": cmp_flops,
                      "rel_error": "rel_error_vs_oracle[<path>_compressed] is against the oracle of the "
                                   "uncompressed method, so it includes the truncation"}
        for name in (args.prec, "fp64", "fp32"):
            if name in compressed:
                continue
            prec = tai.PREC_BY_NAME[name]
            steps = max(1, K // 2)
            log(f"compressed {name}: rank={rank} steps={steps}")
            ms, st, samp = run_steps(prec, B64 if prec == tai.FP64 else B32, steps, 1, Pc)
            a_ms = st["assemble"][0] / max(1, st["assemble"][1])
            compressed[name] = {"ms_per_step": round(ms, 3), "entries_per_s": entries / (ms / 1e3),
                                "stage_ms": stage_ms(st, steps),
                                "assemble_tflops_algorithmic": round(cmp_flops / (a_ms / 1e3) / 1e12, 2)}
            if name in paths:
                compressed[name]["speedup_vs_uncompressed_step"] = round(paths[name]["ms_per_step"] / ms, 3)
                compressed[name]["normwise_change_vs_uncompressed_gpu_sampled"] = float(
                    np.max(np.abs(samp - samples[name])) / np.max(np.abs(samples[name])))
            samples[name + "_compressed"] = samp
        # the second omega of the Nb = 400 workload: omega = 1.0, where the
        # kernel interpolant on [-L, L] is far coarser (the paper notes TA
        # degrades at large omega); the error is reported, not asserted
        b1, P1 = I.spd400(omega=1.0)
        assert np.array_equal(b1.center, b.center) and np.array_equal(b1.alpha, b.alpha)
        omega1 = {"omega": P1.omega, "nq": P1.nq, "n": P1.n, "L": P1.L}
        for name in (args.prec, "fp64", "fp32", "bf16x6"):
            if name in omega1:
                continue
            prec = tai.PREC_BY_NAME[name]
            steps = max(1, K // 2)
            log(f"omega=1.0 {name}: steps={steps}")
            ms, st, samp = run_steps(prec, B64 if prec == tai.FP64 else B32, steps, 1, P1)
            a_ms = st["assemble"][0] / max(1, st["assemble"][1])
            omega1[name] = {"ms_per_step": round(ms, 3), "entries_per_s": entries / (ms / 1e3),
                            "stage_ms": stage_ms(st, steps),
                            "assemble_tflops_algorithmic": round(flops / (a_ms / 1e3) / 1e12, 2)}
            samples_w1[name] = samp
        for name in omega1:
            if isinstance(omega1[name], dict) and "fp64" in omega1:
                omega1[name]["speedup_vs_fp64"] = round(omega1["fp64"]["ms_per_step"] / omega1[name]["ms_per_step"], 3)
        del B64
        torch.cuda.empty_cache()
        if "fp64" in paths:
            for name in paths:
                paths[name]["speedup_vs_fp64"] = round(paths[name]["entries_per_s"] / paths["fp64"]["entries_per_s"], 3)
        for name in ("fp64", "fp32"):
            if name in paths and name in degrees:
                degrees[name]["speedup_vs_fixed_degree"] = round(paths[name]["ms_per_step"] / degrees[name]["ms_per_step"], 3)
        # the assembly kernel of every path against its own arithmetic's peak
        for name, pv in paths.items():
            tf = flops / (pv["stage_ms"]["assemble"] / 1e3) / 1e12
            pv["assemble_tflops_algorithmic"] = round(tf, 2)
            pv["assemble_frac_of_peak"] = round(tf / PEAK_TFLOPS[name], 4)
    del B32
    torch.cuda.empty_cache()

    # ---------------- the Nb = 64 workload: full B in FP64 and FP32 ------------
    small = None
    small_B = {}
    if not args.only_headline:
        b2, P2 = I.sp16()
        ba2 = tai.BasisArrays(b2)
        np2 = b2.npair
        M2 = torch.empty((3, P2.n, np2), dtype=torch.float64, device=dev)
        small = {"workload": f"sp16: Nb={b2.nb} (16 atoms in [-5,5]^3, s+p shells), {np2} pairs, omega={P2.omega}, "
                             f"nq={P2.nq}, n={P2.n}, L={P2.L}; step = moments + full B ({float(np2) * np2:.3g} entries)"}
        for name in ("fp64", "fp32"):
            prec = tai.PREC_BY_NAME[name]
            B2 = torch.empty((np2, np2), dtype=torch.float64 if prec == tai.FP64 else torch.float32, device=dev)
            params2 = tai.make_params(P2, prec)
            log(f"Nb=64 {name}: steps={K}")
            for it in range(W + K):
                if it == W:
                    torch.cuda.synchronize()
                    t0 = time.perf_counter()
                ctx.moments(ba2, P2, M2)
                ctx.assemble_B(M2, np2, params2, B2)
            torch.cuda.synchronize()
            ms2 = (time.perf_counter() - t0) * 1e3 / K
            small[name] = {"ms_per_step": round(ms2, 4), "entries_per_s": float(np2) * np2 / (ms2 / 1e3)}
            small_B[name] = B2.double().cpu().numpy()
            del B2
        small["fp32"]["speedup_vs_fp64"] = round(small["fp64"]["ms_per_step"] / small["fp32"]["ms_per_step"], 3)
        del M2
        torch.cuda.empty_cache()

    # ---------------- the headline step over the pairs kept by screening -------
    screened = None
    screened_sample = None
    adaptive_b_sample = None
    if not args.only_headline:
        pairs = torch.empty(npair, dtype=torch.int32, device=dev)
        params = tai.make_params(P, head)
        Ms = Bs = None
        log(f"screened {args.prec}: tau={SCREEN_TAU}")
        for it in range(W + K):
            if it == W:
                torch.cuda.synchronize()
                ctx.profile_enable(True)
                t0 = time.perf_counter()
            npk = ctx.screen_pairs(ba, SCREEN_TAU, pairs)
            if Ms is None:
                Ms = torch.empty((3, n, npk), dtype=torch.float64, device=dev)
                Bs = torch.empty((npk, npk), dtype=torch.float64 if head == tai.FP64 else torch.float32, device=dev)
            ctx.moments_pairs(ba, P, pairs, npk, Ms)
            ctx.assemble_B(Ms, npk, params, Bs)
        torch.cuda.synchronize()
        ms_s = (time.perf_counter() - t0) * 1e3 / K
        sts = {s_: ctx.profile_read(s_) for s_ in ("moments", "pack", "project", "assemble")}
        ctx.profile_enable(False)
        ent_s = float(npk) * npk
        screened = {"tau": SCREEN_TAU, "kept_pairs": npk, "pairs": npair, "entries": ent_s,
                    "ms_per_step": round(ms_s, 3), "entries_per_s": ent_s / (ms_s / 1e3),
                    "stage_ms": stage_ms(sts, K),
                    "speedup_vs_unscreened_step": round(ms_head / ms_s, 3)}
        ki = rng.integers(0, npk, 240)
        kj = rng.integers(0, npk, 240)
        kept_host = pairs[:npk].cpu().numpy().astype(np.int64)
        screened_sample = (kept_host[ki], kept_host[kj],
                           Bs[torch.as_tensor(ki, device=dev), torch.as_tensor(kj, device=dev)].double().cpu().numpy())
        del Ms, Bs, pairs
        torch.cuda.empty_cache()

    # ---------------- batched persistent assembly (64 molecules) --------------
    batched = None
    if not args.only_headline:
        mols = I.batch64()
        structs, keep, bufs = [], [], []
        for mb, mp in mols:
            bam = tai.BasisArrays(mb)
            Mm = torch.empty((3, mp.n, mb.npair), dtype=torch.float64, device=dev)
            Bm = torch.empty((mb.npair, mb.npair), dtype=torch.float32, device=dev)
            keep.append(bam)
            bufs.append((Mm, Bm))
            structs.append(tai.tai_mol(bam.struct, tai.make_params(mp, head), Mm.data_ptr(), Bm.data_ptr(), mb.npair))
        ent = float(sum(mb.npair ** 2 for mb, _ in mols))
        log("batched: 64 molecules")
        side = torch.cuda.Stream()   # a non-default stream: the batch is replayed from a hipGraph
        torch.cuda.synchronize()
        # the first call tunes the shape and captures the graph; a batch takes
        # ~8 ms, so it is timed over at least 10 replays
        for _ in range(max(W, 3)):
            ctx.assemble_B_batched(structs, stream=side)
        torch.cuda.synchronize()
        kb = max(K, 10)
        t0 = time.perf_counter()
        for _ in range(kb):
            ctx.assemble_B_batched(structs, stream=side)
        torch.cuda.synchronize()
        ms_b = (time.perf_counter() - t0) * 1e3 / kb

        def per_mol():
            for (mb, mp), bam, (Mm, Bm) in zip(mols, keep, bufs):
                ctx.moments(bam, mp, Mm)
                ctx.assemble_B(Mm, mb.npair, tai.make_params(mp, head), Bm)
        for _ in range(W):
            per_mol()
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        for _ in range(K):
            per_mol()
        torch.cuda.synchronize()
        ms_p = (time.perf_counter() - t0) * 1e3 / K
        batched = {"workload": "64 molecules, atoms 5..30 in [-5,5]^3, s+p, omega in {0.3,0.5,1.0}, nq=24, n=32, L=12",
                   "entries": ent, "ms_batched_graph": round(ms_b, 3), "ms_per_molecule_launches": round(ms_p, 3),
                   "entries_per_s_batched": ent / (ms_b / 1e3), "speedup": round(ms_p / ms_b, 3)}
        del bufs
        torch.cuda.empty_cache()

    # ---------------- J through the grid tensor (Nb = 1000) -------------------
    japply = None
    if not args.only_headline:
        jb, jP, D = I.jbuild1000()
        jba = tai.BasisArrays(jb)
        Mj = torch.empty((3, jP.n, jb.npair), dtype=torch.float64, device=dev)
        Dj = torch.as_tensor(D, device=dev)
        JNAMES = ("fp64", "fp32", "bf16x6", "bf16x3")
        Jj = {name: torch.empty((jb.nb, jb.nb), dtype=torch.float64, device=dev) for name in JNAMES}
        japply = {"workload": "Nb=1000 (100 atoms s,p,d), 500500 pairs, omega=0.4, nq=32, n=48, L=24; "
                              "step = moments + J (B never stored)"}
        for name in JNAMES:
            jparams = tai.make_params(jP, tai.PREC_BY_NAME[name])
            log(f"J-build {name}: Nb=1000")
            for _ in range(W):
                ctx.moments(jba, jP, Mj)
                ctx.apply_J(Mj, jb.nb, jparams, Dj, Jj[name])
            torch.cuda.synchronize()
            ctx.profile_enable(True)
            t0 = time.perf_counter()
            for _ in range(K):
                ctx.moments(jba, jP, Mj)
                ctx.apply_J(Mj, jb.nb, jparams, Dj, Jj[name])
            torch.cuda.synchronize()
            ms_j = (time.perf_counter() - t0) * 1e3 / K
            stj = {s_: ctx.profile_read(s_) for s_ in ("moments", "apply_J")}
            ctx.profile_enable(False)
            japply[name] = {"ms_per_step": round(ms_j, 3),
                            "effective_entries_per_s": float(jb.npair) ** 2 / (ms_j / 1e3),
                            "stage_ms": stage_ms(stj, K)}
        # against the oracle: J at 64 sampled pairs by the direct route
        # (J_p = sum_q B(p,q) Dt_q over all 500500 pairs, rows of B from
        # Theorem 3.1), written once by tests/golden/make_jbuild1000.py
        gold = load_j_fixture()
        if gold is not None:
            gp, gj = gold
            gmu = torch.as_tensor(gp[:, 0], device=dev)
            gnu = torch.as_tensor(gp[:, 1], device=dev)
            for name in JNAMES:
                v = Jj[name][gmu, gnu].cpu().numpy()
                japply[name]["rel_2norm_vs_oracle"] = float(np.linalg.norm(v - gj) / np.linalg.norm(gj))
                japply[name]["normwise_vs_oracle"] = float(np.max(np.abs(v - gj)) / np.max(np.abs(gj)))
            japply["oracle_sample"] = (f"{len(gj)} entries J(mu,nu) by the oracle's direct route "
                                       "(tests/golden/jbuild1000_J.json)")
        ref, got = Jj["fp64"], Jj["fp32"]
        japply["fp32"]["rel_2norm_vs_fp64_gpu"] = float(torch.linalg.matrix_norm(got - ref, 2) /
                                                        torch.linalg.matrix_norm(ref, 2))
        japply["fp32"]["normwise_vs_fp64_gpu"] = float((got - ref).abs().max() / ref.abs().max())
        for name in JNAMES[1:]:
            japply[name]["speedup_vs_fp64"] = round(japply["fp64"]["ms_per_step"] / japply[name]["ms_per_step"], 3)
            japply[name]["apply_J_speedup_vs_fp64"] = round(japply["fp64"]["stage_ms"]["apply_J"] /
                                                            japply[name]["stage_ms"]["apply_J"], 3)
        for name in ("bf16x6", "bf16x3"):
            got = Jj[name]
            japply[name]["rel_2norm_vs_fp64_gpu"] = float(torch.linalg.matrix_norm(got - ref, 2) /
                                                          torch.linalg.matrix_norm(ref, 2))
        # the same J-build over the pairs kept by screening
        jpairs = torch.empty(jb.npair, dtype=torch.int32, device=dev)
        jparams = tai.make_params(jP, tai.FP64)
        Js = torch.empty_like(Jj["fp64"])
        Mjs = None
        log(f"screened J-build fp64: tau={SCREEN_TAU}")
        for it in range(W + K):
            if it == W:
                torch.cuda.synchronize()
                ctx.profile_enable(True)
                t0 = time.perf_counter()
            npk_j = ctx.screen_pairs(jba, SCREEN_TAU, jpairs)
            if Mjs is None:
                Mjs = torch.empty((3, jP.n, npk_j), dtype=torch.float64, device=dev)
            ctx.moments_pairs(jba, jP, jpairs, npk_j, Mjs)
            ctx.apply_J_pairs(Mjs, jb.nb, jpairs, npk_j, jparams, Dj, Js)
        torch.cuda.synchronize()
        ms_js = (time.perf_counter() - t0) * 1e3 / K
        stj = {s_: ctx.profile_read(s_) for s_ in ("moments", "apply_J")}
        ctx.profile_enable(False)
        ref = Jj["fp64"]
        screened_j = {"tau": SCREEN_TAU, "kept_pairs": npk_j, "pairs": jb.npair, "ms_per_step": round(ms_js, 3),
                      "stage_ms": stage_ms(stj, K),
                      "speedup_vs_unscreened": round(japply["fp64"]["ms_per_step"] / ms_js, 3),
                      "rel_2norm_vs_unscreened_gpu": float(torch.linalg.matrix_norm(Js - ref, 2) /
                                                           torch.linalg.matrix_norm(ref, 2))}
        japply["screened_fp64"] = screened_j
        # adaptive integration boxes (section 6.2): supports at tau = 1e-20,
        # four equal-count quantile boxes; a step = partitions + moments of
        # every partition on its box + J over the box pairs
        gparts = load_j_fixture("jbuild1000_Jparts.json")
        adaptive = {"tau": PARTS_TAU, "nparts": PARTS_N}
        lst = torch.empty(jb.npair, dtype=torch.int32, device=dev)
        Mpt = torch.empty(3 * jP.n * jb.npair, dtype=torch.float64, device=dev)
        Jpt = torch.empty_like(Jj["fp64"])
        for name in ("fp64", "bf16x6"):
            jparams = tai.make_params(jP, tai.PREC_BY_NAME[name])
            log(f"adaptive-box J-build {name}: nparts={PARTS_N}")
            for it in range(W + K):
                if it == W:
                    torch.cuda.synchronize()
                    ctx.profile_enable(True)
                    t0 = time.perf_counter()
                counts, boxes = ctx.partition_pairs(jba, PARTS_TAU, PARTS_N, lst)
                ctx.moments_partitioned(jba, jP, lst, counts, boxes, Mpt)
                ctx.apply_J_partitioned(Mpt, jb.nb, lst, counts, boxes, jparams, Dj, Jpt)
            torch.cuda.synchronize()
            ms_pt = (time.perf_counter() - t0) * 1e3 / K
            stp = {s_: ctx.profile_read(s_) for s_ in ("nodes", "moments", "apply_J")}
            ctx.profile_enable(False)
            rec = {"ms_per_step": round(ms_pt, 3), "boxes": [round(x, 4) for x in boxes], "counts": counts,
                   "stage_ms": stage_ms(stp, K),
                   "step_ratio_vs_fixed_box": round(ms_pt / japply[name]["ms_per_step"], 3),
                   "rel_2norm_vs_fixed_box_L24_gpu": float(torch.linalg.matrix_norm(Jpt - Jj["fp64"], 2) /
                                                           torch.linalg.matrix_norm(Jj["fp64"], 2))}
            if gparts is not None:
                gp, gj = gparts
                v = Jpt[torch.as_tensor(gp[:, 0], device=dev), torch.as_tensor(gp[:, 1], device=dev)].cpu().numpy()
                rec["rel_2norm_vs_oracle"] = float(np.linalg.norm(v - gj) / np.linalg.norm(gj))
            adaptive[name] = rec
        japply["adaptive_boxes"] = adaptive
        del lst, Mpt, Jpt
        # the same on the Nb = 400 basis (its J with the random density of
        # the J workload's recipe), FP64, against the fixed box L = 16
        b4, P4 = I.spd400(omega=0.3)
        D4 = torch.as_tensor(I.random_density(np.random.default_rng(41), b4), device=dev)
        ba4 = tai.BasisArrays(b4)
        M4 = torch.empty(3 * P4.n * b4.npair, dtype=torch.float64, device=dev)
        J4f = torch.empty((b4.nb, b4.nb), dtype=torch.float64, device=dev)
        J4a = torch.empty_like(J4f)
        lst4 = torch.empty(b4.npair, dtype=torch.int32, device=dev)
        p4 = tai.make_params(P4, tai.FP64)
        log(f"adaptive-box J Nb=400 fp64: nparts={PARTS_N}")
        for it in range(W + K):
            if it == W:
                torch.cuda.synchronize()
                t0 = time.perf_counter()
            ctx.moments(ba4, P4, M4)
            ctx.apply_J(M4, b4.nb, p4, D4, J4f)
        torch.cuda.synchronize()
        ms_f4 = (time.perf_counter() - t0) * 1e3 / K
        for it in range(W + K):
            if it == W:
                torch.cuda.synchronize()
                t0 = time.perf_counter()
            counts4, boxes4 = ctx.partition_pairs(ba4, PARTS_TAU, PARTS_N, lst4)
            ctx.moments_partitioned(ba4, P4, lst4, counts4, boxes4, M4)
            ctx.apply_J_partitioned(M4, b4.nb, lst4, counts4, boxes4, p4, D4, J4a)
        torch.cuda.synchronize()
        ms_a4 = (time.perf_counter() - t0) * 1e3 / K
        adaptive["spd400_fp64"] = {
            "workload": "spd400 basis (Nb=400, 80200 pairs), omega=0.3, nq=32, n=40; J of a random density",
            "boxes": [round(x, 4) for x in boxes4], "counts": counts4,
            "ms_per_step": round(ms_a4, 3), "fixed_box_L16_ms_per_step": round(ms_f4, 3),
            "rel_2norm_vs_fixed_box_L16_gpu": float(torch.linalg.matrix_norm(J4a - J4f, 2) /
                                                    torch.linalg.matrix_norm(J4f, 2))}
        # B over the same four boxes (the stored-matrix form): a step =
        # partitions + moments on the boxes + B, in the headline arithmetic
        # and FP64, against the fixed-box step of the headline workload;
        # sampled entries against Algorithm 1 on the pairs' boxes
        adaptive_b = {"workload": "spd400 basis (Nb=400, 80200 pairs), omega=0.3, nq=32, n=40, four boxes; "
                                  "step = partitions + moments on the boxes + full B (6.43e9 entries)"}
        lst4c = lst4.cpu().numpy().astype(np.int64)
        offs4 = np.concatenate([[0], np.cumsum(counts4)])
        rngb = np.random.default_rng(23)
        bi = np.concatenate([rngb.integers(0, b4.npair, 160), [0, b4.npair - 1]])
        bj = np.concatenate([rngb.integers(0, b4.npair, 160), [b4.npair - 1, 0]])
        for name in (args.prec, "fp64"):
            precb = tai.PREC_BY_NAME[name]
            Bb = torch.empty((npair, ldb), dtype=torch.float64 if precb == tai.FP64 else torch.float32, device=dev)
            pb = tai.make_params(P4, precb)
            log(f"adaptive-box B {name}: nparts={PARTS_N}")
            stepsb = K if precb != tai.FP64 else max(1, K // 2)
            for it in range(1 + stepsb):
                if it == 1:
                    torch.cuda.synchronize()
                    ctx.profile_enable(True)
                    t0 = time.perf_counter()
                counts4, boxes4 = ctx.partition_pairs(ba4, PARTS_TAU, PARTS_N, lst4)
                ctx.moments_partitioned(ba4, P4, lst4, counts4, boxes4, M4)
                ctx.assemble_B_partitioned(M4, counts4, boxes4, pb, Bb, ldb)
            torch.cuda.synchronize()
            ms_b = (time.perf_counter() - t0) * 1e3 / stepsb
            stb = {s_: ctx.profile_read(s_) for s_ in ("nodes", "moments", "pack", "project", "assemble")}
            ctx.profile_enable(False)
            adaptive_b[name] = {"ms_per_step": round(ms_b, 3), "stage_ms": stage_ms(stb, stepsb),
                                "step_ratio_vs_fixed_box": round(ms_b / paths[name]["ms_per_step"], 3),
                                "sample": Bb[torch.as_tensor(bi, device=dev),
                                             torch.as_tensor(bj, device=dev)].double().cpu().numpy()}
            del Bb
            torch.cuda.empty_cache()
        adaptive["spd400_B"] = adaptive_b
        adaptive_b_sample = (lst4c, offs4, list(boxes4), bi, bj)
        del M4, J4f, J4a, lst4
        # the same J-build on the compressed grid (R^3 instead of n^3)
        jPc = dataclasses.replace(jP, rank_tol=RANK_TOL_J)
        ctx.moments(jba, jP, Mj)
        jrank = ctx.compress(Mj, jb.npair, jPc)
        Jc = torch.empty_like(Jj["fp64"])
        for name in ("fp64", "fp32"):
            jparams_c = tai.make_params(jPc, tai.PREC_BY_NAME[name])
            log(f"compressed J-build {name}: rank={jrank}")
            for it in range(W + K):
                if it == W:
                    torch.cuda.synchronize()
                    ctx.profile_enable(True)
                    t0 = time.perf_counter()
                ctx.moments(jba, jP, Mj)
                ctx.apply_J(Mj, jb.nb, jparams_c, Dj, Jc)
            torch.cuda.synchronize()
            ms_jc = (time.perf_counter() - t0) * 1e3 / K
            stj = {s_: ctx.profile_read(s_) for s_ in ("moments", "compress", "apply_J")}
            ctx.profile_enable(False)
            japply["compressed_" + name] = {
                "rank_tol": RANK_TOL_J, "rank": jrank, "n": jP.n, "ms_per_step": round(ms_jc, 3),
                "stage_ms": stage_ms(stj, K),
                "speedup_vs_uncompressed": round(japply[name]["ms_per_step"] / ms_jc, 3),
                "rel_2norm_vs_uncompressed_fp64_gpu": float(torch.linalg.matrix_norm(Jc - Jj["fp64"], 2) /
                                                            torch.linalg.matrix_norm(Jj["fp64"], 2))}
        # with the moments fixed (a self-consistent-field loop changes D only)
        # one compression serves every J build: prepared operands, J alone
        n_j, nq_j = jP.n, jP.nq
        Ub = torch.empty(3 * n_j * jb.npair, dtype=torch.float64, device=dev)
        Kb = torch.empty(nq_j * n_j * n_j, dtype=torch.float64, device=dev)
        ctx.moments(jba, jP, Mj)
        jrank = ctx.compress(Mj, jb.npair, tai.make_params(jPc), U=Ub, Kc=Kb)
        for name in ("fp64", "fp32"):
            jparams_c = tai.make_params(jPc, tai.PREC_BY_NAME[name])
            log(f"J-build from prepared compressed operands {name}: rank={jrank}")
            for it in range(W + K):
                if it == W:
                    torch.cuda.synchronize()
                    t0 = time.perf_counter()
                ctx.apply_J_compressed(Ub, jb.nb, jrank, Kb, jparams_c, Dj, Jc)
            torch.cuda.synchronize()
            ms_p = (time.perf_counter() - t0) * 1e3 / K
            ref_ms = japply[name]["stage_ms"]["apply_J"]
            japply["compressed_" + name]["prepared_ms_per_J"] = round(ms_p, 3)
            japply["compressed_" + name]["prepared_speedup_vs_uncompressed_apply_J"] = round(ref_ms / ms_p, 3)
        del Jc, Ub, Kb
        # the orbital-basis Coulomb matrix of NORB orbitals on the same grid
        Qo = torch.as_tensor(np.random.default_rng(17).standard_normal((NORB, jb.nb)) / np.sqrt(jb.nb), device=dev)
        Jmo = torch.empty((NORB, NORB), dtype=torch.float64, device=dev)
        jparams_mo = tai.make_params(jP, tai.FP64)
        log(f"orbital-basis Coulomb matrix fp64: norb={NORB}")
        ctx.moments(jba, jP, Mj)
        for it in range(W + K):
            if it == W:
                torch.cuda.synchronize()
                t0 = time.perf_counter()
            ctx.coulomb_mo(Mj, jb.nb, jparams_mo, Qo, NORB, Jmo)
        torch.cuda.synchronize()
        ms_mo = (time.perf_counter() - t0) * 1e3 / K
        japply["coulomb_mo_fp64"] = {"norb": NORB, "ms_per_call": round(ms_mo, 3),
                                     "ms_per_orbital": round(ms_mo / NORB, 4),
                                     "symmetry_rel": float((Jmo - Jmo.T).abs().max() / Jmo.abs().max())}
        # the same with the moments compressed on every call (rank_tol > 0):
        # the compression is paid once per call for all NORB orbitals
        jparams_mc = tai.make_params(dataclasses.replace(jP, rank_tol=RANK_TOL_J), tai.FP64)
        Jmo_c = torch.empty_like(Jmo)
        log(f"orbital-basis Coulomb matrix fp64, compressed: norb={NORB} rank_tol={RANK_TOL_J}")
        for it in range(W + K):
            if it == W:
                torch.cuda.synchronize()
                t0 = time.perf_counter()
            ctx.coulomb_mo(Mj, jb.nb, jparams_mc, Qo, NORB, Jmo_c)
        torch.cuda.synchronize()
        ms_mc = (time.perf_counter() - t0) * 1e3 / K
        japply["coulomb_mo_fp64_compressed"] = {
            "norb": NORB, "rank_tol": RANK_TOL_J, "ms_per_call": round(ms_mc, 3),
            "speedup_vs_uncompressed": round(ms_mo / ms_mc, 3),
            "normwise_vs_uncompressed_gpu": float((Jmo_c - Jmo).abs().max() / Jmo.abs().max())}
        # the FP32 pair contraction (the grid sums stay FP64)
        jparams_m32 = tai.make_params(jP, tai.FP32)
        Jmo_32 = torch.empty_like(Jmo)
        log(f"orbital-basis Coulomb matrix fp32: norb={NORB}")
        for it in range(W + K):
            if it == W:
                torch.cuda.synchronize()
                t0 = time.perf_counter()
            ctx.coulomb_mo(Mj, jb.nb, jparams_m32, Qo, NORB, Jmo_32)
        torch.cuda.synchronize()
        ms_m32 = (time.perf_counter() - t0) * 1e3 / K
        japply["coulomb_mo_fp32"] = {
            "norb": NORB, "ms_per_call": round(ms_m32, 3), "speedup_vs_fp64": round(ms_mo / ms_m32, 3),
            "normwise_vs_fp64_gpu": float((Jmo_32 - Jmo).abs().max() / Jmo.abs().max())}
        del Jmo_c, Jmo_32
        del Mj, Jj, Js, Mjs, Jmo
        torch.cuda.empty_cache()
        # the long-range exchange matrix (appendix B) by its factorized form:
        # the X_{j mu} grid tensors over the nb pairs of each mu, the mode
        # products of all (orbital, function) tensors batched, then X Phi^T;
        # on the Nb = 64 workload and on the Nb = 400 headline basis
        norb_x = 8
        exchange = {"norb": norb_x,
                    "flops": "2 n^3 nb^2 norb (X) + norb nb nq 6 n^4 (mode products) + 2 nb^2 norb n^3 (X Phi^T)"}
        for xname, (xb, xP), legs in (("sp16", I.sp16(), ("fp64", "fp32", "fp64_compressed")),
                                      ("spd400", I.spd400(omega=0.3), ("fp64", "fp64_compressed"))):
            xba = tai.BasisArrays(xb)
            Mx = torch.empty((3, xP.n, xb.npair), dtype=torch.float64, device=dev)
            ctx.moments(xba, xP, Mx)
            Qx = torch.as_tensor(np.random.default_rng(19).standard_normal((norb_x, xb.nb)) / np.sqrt(xb.nb),
                                 device=dev)
            Kx = torch.empty((xb.nb, xb.nb), dtype=torch.float64, device=dev)
            nx, nqx, nbx = xP.n, xP.nq, xb.nb
            xfl = 2.0 * nx ** 3 * nbx ** 2 * norb_x + norb_x * nbx * nqx * 6.0 * nx ** 4 + 2.0 * nbx ** 2 * norb_x * nx ** 3
            rec = {"workload": f"{xname}: Nb={nbx}, {xb.npair} pairs, nq={nqx}, n={nx}, {norb_x} orbitals",
                   "tensors": norb_x * nbx, "flops_per_call": xfl}
            Kx64 = None
            for name in legs:
                # the Nb = 64 leg at the J legs' tolerance, the Nb = 400 leg at
                # the B legs' (its grid rank, 31 of 40, pads to 32)
                tol_x = RANK_TOL_J if xname == "sp16" else RANK_TOL
                Px = dataclasses.replace(xP, rank_tol=tol_x) if name.endswith("compressed") else xP
                prec = tai.FP32 if name == "fp32" else tai.FP64
                xparams = tai.make_params(Px, prec)
                kx = K if xname == "sp16" else max(1, K // 2)
                log(f"exchange {xname} {name}: Nb={nbx} norb={norb_x} calls={kx}")
                for it in range(W + kx):
                    if it == W:
                        torch.cuda.synchronize()
                        ctx.profile_enable(True)
                        t0 = time.perf_counter()
                    ctx.exchange(Mx, nbx, xparams, Qx, norb_x, Kx)
                torch.cuda.synchronize()
                ms_x = (time.perf_counter() - t0) * 1e3 / kx
                kern = ctx.profile_read("apply_J")
                ctx.profile_enable(False)
                kms = kern[0] / kx
                rec[name] = {"ms_per_call": round(ms_x, 3), "kernels_ms": round(kms, 3),
                             "symmetry_rel": float((Kx - Kx.T).abs().max() / Kx.abs().max())}
                if name == "fp64":
                    Kx64 = Kx.clone()
                elif Kx64 is not None:
                    rec[name]["normwise_vs_fp64_gpu"] = float((Kx - Kx64).abs().max() / Kx64.abs().max())
                    if name.endswith("compressed"):
                        rec[name]["rank_tol"] = tol_x
                        rec[name]["speedup_vs_fp64"] = round(rec["fp64"]["ms_per_call"] / ms_x, 3)
                if name == "fp64":
                    tf = xfl / (kms / 1e3) / 1e12
                    rec[name]["tflops_algorithmic"] = round(tf, 2)
                    # the fraction of the peak counts what is issued: up to
                    # n = 32 the tables' mirror symmetry leaves half of the
                    # mode products (k_phi.hip)
                    saved = norb_x * nbx * nqx * 3.0 * nx ** 4 if nx <= 32 else 0.0
                    rec[name]["frac_of_fp64_peak"] = round(tf * (1.0 - saved / xfl) / PEAK_TFLOPS["fp64"], 4)
            exchange[xname] = rec
            del Mx, Kx, Kx64
            torch.cuda.empty_cache()
        japply["exchange"] = exchange

    # ---------------- the device's own sustained peaks ------------------------
    if not args.only_headline:
        log("peak probes")
        ach = {"mfma_f16_tflops": round(ctx.peak_probe(0), 1), "mfma_f64_tflops": round(ctx.peak_probe(1), 2),
               "hbm_copy_gbs": round(ctx.peak_probe(2), 0)}
        roofline["achievable"] = ach
        key = {"fp64": "mfma_f64_tflops", "fp32": None}.get(args.prec, "mfma_f16_tflops")
        if key:
            roofline["frac_of_achievable"] = round(achieved / ach[key], 5)

    # ---------------- oracle on the host (bounded sample) ---------------------
    cpu = None
    rel_error = None
    if not args.no_cpu:
        from oracle import tairef as T
        try:
            from threadpoolctl import threadpool_info
            cores = max([x.get("num_threads", 1) for x in threadpool_info()] + [1])
        except Exception:
            cores = os.cpu_count()
        log(f"oracle sample on the host ({cores} threads)")
        sel = np.unique(np.concatenate([sp, sq]))
        cols_extra = rng.choice(npair, 14000, replace=False)
        allp = np.unique(np.concatenate([sel, cols_extra]))
        # the sample: oracle moments of `allp` and a block of B rows against all
        # of them; the row count is sized from a short probe so that the timed
        # oracle work takes about args.cpu_seconds
        t0 = time.perf_counter()
        Mr = T.moments(b.center, b.alpha, b.lxyz, P.L, P.n, pairs=allp)
        t, w = T.time_nodes(P.omega, P.nq)
        xi, _ = T.cheb_nodes(P.n, P.L)
        Kt = T.ktables(t, xi)
        t_mom = time.perf_counter() - t0
        tp = time.perf_counter()
        T.B_full(Mr, Kt, w, rows=np.arange(64))
        per_row = (time.perf_counter() - tp) / 64
        nrows = int(min(len(allp), max(16, (args.cpu_seconds - t_mom) / max(per_row, 1e-6))))
        rows = np.sort(rng.choice(len(allp), nrows, replace=False))
        tb = time.perf_counter()
        Brows = T.B_full(Mr, Kt, w, rows=rows)
        t_or = t_mom + (time.perf_counter() - tb)
        n_or = Brows.size
        cpu = {"value": n_or / t_or, "unit": "entries/s", "cores": int(cores), "kind": "oracle",
               "sample": f"moments of {len(allp)} sampled pairs + B on {len(rows)} x {len(allp)} entries "
                         f"(Theorem 3.1 matrix route) of the Nb=400 workload, {t_or:.1f} s of oracle work"}
        ref = T.B_entries(Mr, Kt, w, np.searchsorted(allp, sp), np.searchsorted(allp, sq))
        dref = T.B_entries(Mr, Kt, w, np.searchsorted(allp, sel), np.searchsorted(allp, sel))
        scale = float(np.max(np.abs(dref)))
        rel_error = {}
        ref_deg = None
        if degrees is not None:
            Ktr = T.truncated_tables(t, xi, P.L, DEGREE_TOL)[2]
            ref_deg = T.B_entries(Mr, Ktr, w, np.searchsorted(allp, sp), np.searchsorted(allp, sq))
            degrees["oracle_change_vs_fixed_degree"] = float(np.max(np.abs(ref_deg - ref)) / scale)
        if screened_sample is not None:
            gi, gj, sv = screened_sample
            allk = np.unique(np.concatenate([gi, gj]))
            Mk = T.moments(b.center, b.alpha, b.lxyz, P.L, P.n, pairs=allk)
            ref_s = T.B_entries(Mk, Kt, w, np.searchsorted(allk, gi), np.searchsorted(allk, gj))
            err = np.abs(sv - ref_s)
            rel_error[args.prec + "_screened"] = {"normwise": float(np.max(err) / scale)}
        def errors(sv, r, scale_):
            err = np.abs(sv - r)
            big_ = np.abs(r) >= 1e-8 * scale_
            mid_ = np.abs(r) >= 1e-4 * scale_
            return {"normwise": float(np.max(err) / scale_),
                    "frobenius_sampled": float(np.linalg.norm(sv - r) / np.linalg.norm(r)),
                    "elementwise_mean": float(np.mean(err[big_] / np.abs(r[big_]))),
                    "elementwise_max": float(np.max(err[big_] / np.abs(r[big_]))),
                    "elementwise_max_above_1e-4": float(np.max(err[mid_] / np.abs(r[mid_])))}

        for name, sv in samples.items():
            rel_error[name] = errors(sv, ref_deg if name.endswith("_degrees") else ref, scale)
        # omega = 1.0: the same moments, the nodes and tables of omega = 1.0
        if samples_w1:
            t1, w1 = T.time_nodes(1.0, P.nq)
            Kt1 = T.ktables(t1, xi)
            ref1 = T.B_entries(Mr, Kt1, w1, np.searchsorted(allp, sp), np.searchsorted(allp, sq))
            scale1 = float(np.max(np.abs(T.B_entries(Mr, Kt1, w1, np.searchsorted(allp, sel),
                                                      np.searchsorted(allp, sel)))))
            omega1["rel_error_vs_oracle"] = {name: errors(sv, ref1, scale1) for name, sv in samples_w1.items()}
        # B over the four boxes of the Nb = 400 basis: the oracle's moments
        # of the sampled pairs on their boxes, Algorithm 1 on the pairs' boxes
        if adaptive_b_sample is not None:
            order4, offs4, boxes4, bi, bj = adaptive_b_sample
            part_of = np.searchsorted(offs4, np.arange(len(order4)), side="right") - 1
            t4, w4 = T.time_nodes(P4.omega, P4.nq)
            used = np.unique(np.concatenate([bi, bj]))
            pm4 = []
            for s_ in range(len(boxes4)):
                pos = used[part_of[used] == s_]
                sel4 = order4[pos]
                o_ = np.argsort(sel4)
                sel4 = sel4[o_]
                Ms = (T.moments(b4.center, b4.alpha, b4.lxyz, boxes4[s_], P4.n, pairs=sel4) if len(sel4)
                      else np.zeros((3, P4.n, 0)))
                pm4.append((sel4, Ms))
            ref4 = T.B_partitioned_entries(pm4, boxes4, t4, w4, P4.n, order4[bi], order4[bj])
            scale4 = float(np.max(np.abs(T.B_partitioned_entries(pm4, boxes4, t4, w4, P4.n, order4[used],
                                                                 order4[used]))))
            for name in list(japply["adaptive_boxes"]["spd400_B"]):
                rec_b = japply["adaptive_boxes"]["spd400_B"][name]
                if isinstance(rec_b, dict) and "sample" in rec_b:
                    rec_b["rel_error_vs_oracle"] = errors(rec_b.pop("sample"), ref4, scale4)
        # Nb = 64: every entry of B against the oracle's B (Theorem 3.1 matrix route)
        if small_B:
            Mo = T.moments(b2.center, b2.alpha, b2.lxyz, P2.L, P2.n)
            t2, w2 = T.time_nodes(P2.omega, P2.nq)
            xi2, _ = T.cheb_nodes(P2.n, P2.L)
            Bo = T.B_full(Mo, T.ktables(t2, xi2), w2)
            so = float(np.max(np.abs(Bo)))
            for name, Bg in small_B.items():
                e = errors(Bg, Bo, so)
                e["frobenius"] = e.pop("frobenius_sampled")
                small[name]["rel_error_vs_oracle"] = e
        # the same oracle B rows on one thread (moments excluded on both sides)
        b_rate = Brows.size / (t_or - t_mom)
        try:
            from threadpoolctl import threadpool_limits
            rows1 = rows[:32]
            with threadpool_limits(1):
                t1s = time.perf_counter()
                T.B_full(Mr, Kt, w, rows=rows1)
                t1s = time.perf_counter() - t1s
            cpu["single_thread"] = {"value": len(rows1) * len(allp) / t1s, "unit": "entries/s", "cores": 1,
                                    "sample": f"B on {len(rows1)} x {len(allp)} entries, moments excluded, "
                                              f"{t1s:.1f} s",
                                    "b_only_value_all_threads": b_rate}
        except ImportError:
            pass

    # samples the oracle did not see (--no-cpu) do not go into the line
    if japply is not None and "spd400_B" in japply.get("adaptive_boxes", {}):
        for rec_b in japply["adaptive_boxes"]["spd400_B"].values():
            if isinstance(rec_b, dict):
                rec_b.pop("sample", None)
    out = {
        "metric": METRIC,
        "value": value,
        "unit": "entries/s",
        "n_gpus": 1,
        "steps": K,
        "warmup": W,
        "ms_per_step": round(ms_head, 3),
        "higher_is_better": True,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": args.prec,
        "data": "synthetic",
        "config": {"workload": "spd400: Nb=400 (40 atoms in [-8,8]^3, s+p+d shells), 80200 pairs, "
                               "omega=0.3, nq=32, n=40, L=16; step = moments + full B (6.43e9 entries)",
                   "nb": b.nb, "npair": npair, "entries": entries, "omega": P.omega, "nq": nq, "n": n, "L": P.L,
                   "ldb": ldb, "parallelism": "single GPU"},
        "roofline": roofline,
        "cpu_baseline": cpu,
        "rel_error_vs_oracle": rel_error,
        "paths": paths,
        "degrees": degrees,
        "compressed": compressed,
        "screened": screened,
        "batched": batched,
        "omega_1": omega1,
        "nb64": small,
        "japply": japply,
    }
    print(json.dumps(out), flush=True)


if __name__ == "__main__":
    main()
