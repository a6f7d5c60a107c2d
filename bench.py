"""Benchmark of the energy-based FEM hot path on one MI355X.

Workload (the throughput configuration): unit cube, 64^3 hexes split into six
tetrahedra each (1,572,864 Tet4, 274,625 nodes, 823,875 DOF), compressible
neo-Hookean mu = 1, lam = 1.5, linearization point u = 0.00125 N(0,1) (seed 0),
100 unit directions (seeds 100..199) resident in HBM.  One step = one
linearization plus 100 FP64 tangent actions y = K(u) v (efem_hvp).  `value` is
DOF/s of the tangent action over the timed steps.

Beside it: the FP32 tangent action, the colour and atomic scatters, energy
and residual times, the same operators under the small-strain linear model,
the non-variational transport operator with a GMRES solve, the 2D Tri3
plane-strain tangent action (1024^2 cells), the Hex8 tangent action of the
96^3 and 128^3 compression meshes (FP64 and FP32, %VALU and %HBM), a roofline
object for the dominant kernel (the FP64 tangent action's chunk pass with its
halo gather, over the step's 100 directions, timed with HIP events on its
stream), the Newton
solves of the metric's second half (plain FP64 Jacobi-CG vs FP32 tangent
actions with and without the learned preconditioner, on the 128^3 Q1-hex
compression case and on the unseen 96^3 test mesh of the preconditioner,
the network trained first in the energy norm on CG residuals from 32^3
solves), and the FP64 CPU oracle timed on a bounded sample on the host cores.

    python bench.py [--gpus 1] [--steps K] [--warmup W] [--no-solve] [--no-cpu]
    python bench.py --mode kernels     # fixed kernel workload for rocprofv3
"""
from __future__ import annotations

import argparse
import json
import os
import sys
import time

import numpy as np

ROOT = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, ROOT)

HBM_PEAK_GBS = 8000.0
FP64_PEAK_TFLOPS = 78.6      # MI355X FP64 vector
N_DIRS = 100
# FP64 operations of the Tet4 tangent action in the formulation the kernels
# evaluate (an FMA counts 2, a reciprocal or logarithm 1).  One tetrahedron on
# its own: gradients 27, two adjugates with determinants 64, S = Ae Ae^T 30
# and its scale 6, scalars 14 (two reciprocals, ln J), W = Ad dJ 45, trace
# and coefficients 5, V = cW + bI 12, Q = dJ S + (V Ad)^T 99, the fourth
# node's force 6, the scatter adds 12: 320.  A face pair (two of them) shares
# two gradient edges of each field (18), the adjugates' last rows (18), S22
# (5) and two entries of W (10), and its forces take 6 fewer: 583.
FLOPS_PER_TET_HVP = 320
FLOPS_PER_PAIR_HVP = 2 * FLOPS_PER_TET_HVP - 18 - 18 - 5 - 10 - 6
# One Hex8 tangent action (2x2x2 Gauss) on four lanes, one x-edge and two
# points each, as both precisions evaluate it: per lane 25 flops a component
# for the gradients of each of X, x (or u) and v and 30 a component for the
# forces; per point the arithmetic of a tetrahedron without its gradients and
# forces, 275: 3,460 per hexahedron.
FLOPS_PER_HEX_HVP = 4 * (3 * 3 * 25 + 3 * 30) + 8 * 275


def tet4_hvp_alg(n_elems, n_nodes, n_items):
    """Algorithmic HBM bytes and FP64 operations of one FP64 Tet4 tangent
    action (Eq. 3): int32 connectivity (16 bytes per tetrahedron), X, x and v
    read and y written (24 bytes per node each); FLOPS_PER_PAIR_HVP per face
    pair and FLOPS_PER_TET_HVP per single tetrahedron (n_items work items,
    each a pair or a single)."""
    n_pairs = n_elems - n_items
    alg_bytes = n_elems * 4 * 4 + 4 * n_nodes * 3 * 8
    alg_flops = n_pairs * FLOPS_PER_PAIR_HVP + (n_elems - 2 * n_pairs) * FLOPS_PER_TET_HVP
    return alg_bytes, alg_flops


def roofline_bound(alg_bytes, alg_flops):
    """The bound of a kernel: the longer of its two ideal times at the MI355X
    peaks, alg_bytes / 8 TB/s ("hbm") or alg_flops / 78.6 TFLOP/s ("alu")."""
    return "hbm" if alg_bytes / (HBM_PEAK_GBS * 1e9) >= alg_flops / (FP64_PEAK_TFLOPS * 1e12) else "alu"


def log(msg):
    print(f"[bench] {msg}", file=sys.stderr, flush=True)


def event_time(fn, reps, stream):
    import torch
    start = torch.cuda.Event(enable_timing=True)
    end = torch.cuda.Event(enable_timing=True)
    torch.cuda.synchronize()
    start.record(stream)
    for _ in range(reps):
        fn()
    end.record(stream)
    torch.cuda.synchronize()
    return start.elapsed_time(end) / 1e3 / reps   # seconds per call


COUNTERS_MD = os.path.join(ROOT, "profiles", "hvp_tet4_f64_64cube_counters.md")


def kernel_source_hash():
    """Hash of the element-kernel sources with comments and whitespace taken
    out; counter summaries record it so that stale HBM-traffic figures are
    not reported for a changed kernel (a comment edit changes no kernel)."""
    import hashlib
    import re
    h = hashlib.sha256()
    for name in ("kernels.hip", "efem_internal.h"):
        with open(os.path.join(ROOT, "paper_2602_12365_amd", "csrc", name)) as f:
            src = f.read()
        src = re.sub(r"/\*.*?\*/", " ", src, flags=re.S)   # block comments
        src = re.sub(r"//[^\n]*", " ", src)                 # line comments
        h.update("".join(src.split()).encode())
    return h.hexdigest()[:16]


def measured_traffic():
    """HBM bytes of one FP64 tangent action (block pass + halo gather) from
    the committed rocprofv3 counter summary, or None if it is missing or was
    taken on different kernel sources."""
    try:
        with open(COUNTERS_MD) as f:
            lines = f.read().splitlines()
    except OSError:
        return None
    vals = {}
    for line in lines:
        if line.startswith("- ") and ": " in line:
            k, v = line[2:].split(": ", 1)
            vals[k.strip("` ")] = v.strip("` ")
    if vals.get("kernel_source_hash") != kernel_source_hash():
        return None
    try:
        return int(vals["traffic_bytes_per_launch"])
    except (KeyError, ValueError):
        return None


def solve_section(args, dev):
    """Compression load case (bottom clamped, top -20% z in 10 load steps, Q1
    hexes, 2x2x2 Gauss, mu ~ lognormal(0, 0.5), lam = 1.5 mu) on the 128^3
    mesh (mu seed 3) and on the unseen 96^3 test mesh of the preconditioner
    (mu seed 2000): plain FP64 Newton-CG (Jacobi), mixed FP32-HVP (Jacobi), and
    mixed FP32-HVP with the learned preconditioner trained on 32^3 samples,
    for the first 8 flexible-CG iterations of each Krylov solve (then Jacobi
    PCG from that iterate) and, beside it, for whole solves.
    Wall time from the first load step to the last step's convergence."""
    import torch
    from paper_2602_12365_amd import Operator, inputs as I, precond as PC

    res = {}
    t0 = time.time()
    seeds = range(1000, 1000 + args.train_fields)
    S = PC.generate_samples(n=args.n_train, seeds=seeds, n_steps=10, log=log)
    torch.cuda.synchronize()
    t_samples = time.time() - t0
    t0 = time.time()
    theta, hist = PC.train_energy(S, epochs=args.epochs, lr=args.lr, log=log)
    torch.cuda.synchronize()
    t_train = time.time() - t0
    res["training"] = {"mesh": f"{args.n_train}^3 Q1 hexes", "fields": len(seeds), "load_steps": 10,
                       "samples": S.n_samples, "rows": int(S.X.shape[0]), "epochs": args.epochs,
                       "objective": "energy norm sum_s w_s (z.Kz - 2 r.z), w_s = 1/(S r.D^-1 r)",
                       "objective_jacobi_trained": [hist[0][1], hist[-1][1]],
                       "sample_generation_s": round(t_samples, 2), "training_s": round(t_train, 2)}
    for st in S.states:
        st[0].close()
    del S

    # the configured variant: 200 (residual, Newton correction) pairs (20 fields
    # x 10 load steps on 32^3), the relative target fit of the first version
    theta_pairs = None
    if args.n_test > 0:
        t0 = time.time()
        Xp, auxp, opp = PC.generate_rows(n=args.n_train, seeds=seeds, n_steps=10, log=log)
        torch.cuda.synchronize()
        t_pairs = time.time() - t0
        t0 = time.time()
        theta_pairs, hist_p = PC.train(opp, Xp, auxp, epochs=400, lr=3e-3, log=log)
        torch.cuda.synchronize()
        res["training_pairs"] = {"mesh": f"{args.n_train}^3 Q1 hexes", "fields": len(seeds), "load_steps": 10,
                                 "pairs": len(seeds) * 10, "rows": int(Xp.shape[0]), "epochs": 400,
                                 "objective": "relative target fit |M(-r) - delta|^2/|delta|^2, delta = K^-1(-r)",
                                 "loss_first_last": [hist_p[0][1], hist_p[-1][1]],
                                 "pair_generation_s": round(t_pairs, 2), "training_s": round(time.time() - t0, 2)}
        opp.close()
        del Xp, auxp

    res["solves"] = {}
    for tag, n, seed in (("cfg3", args.n_cfg3, 3), ("cfg5_test", args.n_test, 2000)):
        if n <= 0:
            continue
        res["solves"][tag] = compression_solves(dev, n, seed, theta,
                                                theta_pairs if tag == "cfg5_test" else None)
    # the metric's headline pair: plain FP64 vs mixed FP32 + learned, and mixed
    # FP32 + Jacobi, on the largest configuration run
    main = res["solves"].get("cfg3") or res["solves"].get("cfg5_test")
    runs = main["runs"]
    res["speedup_mixed_learned_vs_plain"] = round(runs["plain_f64_jacobi"]["wall_s"]
                                                  / runs["mixed_f32_learned"]["wall_s"], 3)
    res["speedup_mixed_jacobi_vs_plain"] = round(runs["plain_f64_jacobi"]["wall_s"]
                                                 / runs["mixed_f32_jacobi"]["wall_s"], 3)
    # what the network itself gains: learned against Jacobi at the same
    # (mixed) precision (below 1: the network costs more than it saves)
    res["speedup_learned_vs_mixed_jacobi"] = round(runs["mixed_f32_jacobi"]["wall_s"]
                                                   / runs["mixed_f32_learned"]["wall_s"], 3)
    # the fastest classical preconditioner at both precisions
    res["speedup_mixed_block_vs_plain_block"] = main["speedup_mixed_block_vs_plain_block"]
    return res


def compression_solves(dev, n, seed, theta, theta_pairs=None):
    """Compression case on n^3 Q1 hexes (mu seed `seed`): plain FP64 Jacobi,
    mixed FP32 Jacobi, mixed FP32 with the learned preconditioner (8
    flexible-CG iterations per Krylov solve, and whole solves), and 3x3 block
    Jacobi at both precisions."""
    import torch
    from paper_2602_12365_amd import Operator, inputs as I, precond as PC
    mesh, mu, lam, mask, ubc = PC.compression_case(I.HEX8, n, seed)
    res = {"load_case": f"{n}^3 Q1 hexes ({mesh.n_dofs} DOF), mu~lognormal(0,0.5) seed {seed}, "
                        f"lam=1.5mu, top -20% z in 10 steps, stop at 1e-8 relative residual per step"}
    op = Operator(I.HEX8, mesh.X, mesh.conn, device=dev)
    op.set_material(torch.as_tensor(mu, device=dev), torch.as_tensor(lam, device=dev))
    op.set_dirichlet(torch.as_tensor(mask, device=dev))
    ubc_t = torch.as_tensor(ubc, device=dev)
    op.set_mlp(theta)
    runs = {}
    u_ref = None
    plan = [("plain_f64_jacobi", dict(hvp_prec="f64", precond=0)),
            ("mixed_f32_jacobi", dict(hvp_prec="f32", precond=0)),
            ("mixed_f32_learned", dict(hvp_prec="f32", precond=1, learned_iters=8)),
            ("mixed_f32_learned_whole_solve", dict(hvp_prec="f32", precond=1, learned_iters=0)),
            # 3x3 block Jacobi: the inverses of the nodes' diagonal blocks of K_ff
            ("plain_f64_block_jacobi", dict(hvp_prec="f64", precond=2)),
            ("mixed_f32_block_jacobi", dict(hvp_prec="f32", precond=2))]
    if theta_pairs is not None:
        plan += [("mixed_f32_learned_pairs", dict(hvp_prec="f32", precond=1, learned_iters=8, theta=theta_pairs)),
                 ("mixed_f32_learned_pairs_whole_solve",
                  dict(hvp_prec="f32", precond=1, learned_iters=0, theta=theta_pairs))]
    for name, kw in plan:
        kw = dict(kw)
        op.set_mlp(kw.pop("theta", theta))
        u = torch.zeros((mesh.n_nodes, 3), dtype=torch.float64, device=dev)
        log(f"solve {name}")
        torch.cuda.synchronize()
        t0 = time.time()
        rc, st = op.newton_solve(u, ubc_t, n_steps=10, **kw)
        torch.cuda.synchronize()
        wall = time.time() - t0
        r = op.residual(u)
        entry = {"rc": rc, "wall_s": round(wall, 3), "solver_s": round(st["seconds"], 3),
                 "newton_iters": st["newton_iters"], "cg_iters": st["cg_iters"],
                 "fallbacks": st["precond_fallbacks"], "final_residual_fp64": st["final_residual"],
                 "newton_per_step": st["newton_per_step"], "cg_per_step": st["cg_per_step"],
                 "energy": st["final_energy"]}
        if kw["precond"] == 1:
            # flexible-CG iterations with the network before Jacobi PCG takes over (0: all)
            entry["learned_iters"] = kw["learned_iters"]
        if u_ref is None:
            u_ref = u.clone()
        else:
            entry["rel_diff_to_plain_f64"] = float(torch.linalg.norm(u - u_ref) / torch.linalg.norm(u_ref))
        entry["residual_norm_check"] = float(torch.linalg.norm(r))
        runs[name] = entry
        log(f"{name}: {entry['wall_s']} s, newton {entry['newton_iters']}, cg {entry['cg_iters']}")
    res["runs"] = runs
    res["speedup_mixed_learned_vs_plain"] = round(runs["plain_f64_jacobi"]["wall_s"]
                                                  / runs["mixed_f32_learned"]["wall_s"], 3)
    res["speedup_mixed_jacobi_vs_plain"] = round(runs["plain_f64_jacobi"]["wall_s"]
                                                 / runs["mixed_f32_jacobi"]["wall_s"], 3)
    res["speedup_learned_vs_mixed_jacobi"] = round(runs["mixed_f32_jacobi"]["wall_s"]
                                                   / runs["mixed_f32_learned"]["wall_s"], 3)
    res["speedup_mixed_block_vs_plain_block"] = round(runs["plain_f64_block_jacobi"]["wall_s"]
                                                      / runs["mixed_f32_block_jacobi"]["wall_s"], 3)
    res["speedup_mixed_block_vs_plain_jacobi"] = round(runs["plain_f64_jacobi"]["wall_s"]
                                                       / runs["mixed_f32_block_jacobi"]["wall_s"], 3)
    op.close()
    return res


def kernels_mode(args, dev):
    """Fixed kernel workload for rocprofv3 (no timing logic): the FP64 and FP32
    tangent actions (chunk pass + halo gather) on the 64^3 Kuhn mesh, energy,
    residual, and a plain 256 MiB device copy of known size that calibrates
    the HBM counters.  --flush: a 512 MiB fill before every FP64 tangent
    action, so that its counters see the 256 MB Infinity Cache cold."""
    import torch
    from paper_2602_12365_amd import Operator, inputs as I
    if args.kernels_elem == "hex8":
        return hex8_kernels_mode(args, dev)
    mesh = I.tet_mesh(args.n)
    u = torch.as_tensor(I.gaussian_field(mesh.n_nodes, I.cube_amplitude(args.n), 0)).to(dev)
    v = torch.as_tensor(I.unit_direction(mesh.n_nodes, 100)).to(dev)
    y = torch.zeros_like(u)
    op = Operator(I.TET4, mesh.X, mesh.conn, device=dev)
    op.linearize(u, "f64")
    flush = torch.empty(512 << 20, dtype=torch.uint8, device=dev) if args.flush else None
    for _ in range(args.steps):
        if flush is not None:
            flush.fill_(1)
        op.hvp_zeroed(v, y)
    del flush
    op.linearize(u, "f32")
    v32, y32 = v.float(), torch.zeros_like(v, dtype=torch.float32)
    for _ in range(args.steps):
        op.hvp_zeroed(v32, y32)
    psi = torch.empty((), dtype=torch.float64, device=dev)
    for _ in range(args.steps):
        op.energy(u, out=psi)
        op.residual(u, out=y)
    a = torch.empty(256 << 20, dtype=torch.uint8, device=dev)
    b = torch.empty_like(a)
    for _ in range(5):
        b.copy_(a)
    torch.cuda.synchronize()
    log("kernels mode done")


def hex8_kernels_mode(args, dev):
    """Fixed Hex8 kernel workload for rocprofv3: the FP64 and FP32 tangent
    actions of one compression mesh (n^3 Q1 hexes, mu lognormal(0, 0.5),
    seed 2000 at n = 96 and 3 otherwise, lam = 1.5 mu), --steps calls each."""
    import torch
    from paper_2602_12365_amd import Operator, inputs as I
    n = args.n
    m = I.hex_mesh(n)
    mu = torch.as_tensor(I.lognormal_field(m.n_elems, 0.5, 2000 if n == 96 else 3)).to(dev)
    op = Operator(I.HEX8, m.X, m.conn, device=dev)
    op.set_material(mu, 1.5 * mu)
    u = torch.as_tensor(I.gaussian_field(m.n_nodes, I.cube_amplitude(n), 0)).to(dev)
    v = torch.as_tensor(I.unit_direction(m.n_nodes, 100)).to(dev)
    for prec, dt in (("f64", torch.float64), ("f32", torch.float32)):
        op.linearize(u, prec)
        vv = v.to(dt)
        y = torch.zeros_like(vv)
        for _ in range(args.steps):
            op.hvp_zeroed(vv, y)
    torch.cuda.synchronize()
    op.close()
    log(f"hex8 kernels mode n={n} done")


def hex8_section(args, dev, stream):
    """The Hex8 tangent action (Q1, 2x2x2 Gauss) of the compression meshes:
    96^3 (mu lognormal(0, 0.5) seed 2000, the preconditioner's test mesh) and
    128^3 (seed 3), lam = 1.5 mu, at u = 0.01 (8/n) N(0,1): FP64 and FP32 per
    call over 20 distinct directions, with %HBM of the algorithmic bytes
    (connectivity 32 B/hex, mu and lam 16 B/hex, X, x and v read and y written
    per node) and %VALU of the counted FP64 operations (FLOPS_PER_HEX_HVP)
    against the 78.6 TFLOP/s vector peak."""
    import torch
    from paper_2602_12365_amd import Operator, inputs as I
    res = {"flops_per_hex": FLOPS_PER_HEX_HVP,
           "note": "%VALU = counted FP64 operations / time / 78.6 TFLOP/s (FP32 without packed math has the same issue rate)"}
    for n, seed in ((96, 2000), (128, 3)):
        if (n == 96 and args.n_test == 0) or (n == 128 and args.n_cfg3 == 0):
            continue
        m = I.hex_mesh(n)
        mu = torch.as_tensor(I.lognormal_field(m.n_elems, 0.5, seed)).to(dev)
        op = Operator(I.HEX8, m.X, m.conn, device=dev)
        op.set_material(mu, 1.5 * mu)
        u = torch.as_tensor(I.gaussian_field(m.n_nodes, I.cube_amplitude(n), 0)).to(dev)
        dirs = [torch.as_tensor(I.unit_direction(m.n_nodes, 100 + k)).to(dev) for k in range(20)]
        row = {"mesh": f"{n}^3 Q1 hexes: {m.n_elems} Hex8, {m.n_nodes} nodes, {m.n_dofs} DOF"}
        flops = m.n_elems * FLOPS_PER_HEX_HVP
        for prec, dt, word in (("f64", torch.float64, 8), ("f32", torch.float32, 4)):
            op.linearize(u, prec)
            vv = [d.to(dt) for d in dirs]
            y = torch.empty_like(vv[0])
            op.hvp(vv[0], out=y)

            def sweep():
                for d in vv:
                    op.hvp(d, out=y)
            t = event_time(sweep, 5, stream) / len(vv)
            byts = m.n_elems * (32 + 16) + 4 * m.n_nodes * 3 * word
            row[prec] = {"us": round(t * 1e6, 2), "gdofs": round(m.n_dofs / t / 1e9, 3),
                         "alg_bytes": byts, "pct_hbm": round(100 * byts / t / 1e9 / HBM_PEAK_GBS, 2),
                         "tflops": round(flops / t / 1e12, 3),
                         "pct_valu": round(100 * flops / t / 1e12 / FP64_PEAK_TFLOPS, 2)}
            log(f"hex8 {n}^3 {prec}: {t*1e6:.1f} us, {row[prec]['pct_valu']}% VALU, {row[prec]['pct_hbm']}% HBM")
        res[f"n{n}"] = row
        op.close()
        del dirs, u, mu
    return res


def main():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=20)
    ap.add_argument("--warmup", type=int, default=3)
    ap.add_argument("--n", type=int, default=64, help="hexes per cube edge")
    ap.add_argument("--n2d", type=int, default=1024, help="cells per edge of the 2D Tri3 mesh")
    ap.add_argument("--cpu-seconds", type=float, default=10.0)
    ap.add_argument("--no-cpu", action="store_true")
    ap.add_argument("--no-solve", action="store_true")
    ap.add_argument("--n-train", type=int, default=32)
    ap.add_argument("--n-test", type=int, default=96, help="learned-preconditioner test mesh (0 = skip)")
    ap.add_argument("--n-cfg3", type=int, default=128, help="compression-solve mesh (0 = skip)")
    ap.add_argument("--train-fields", type=int, default=20)
    ap.add_argument("--epochs", type=int, default=300)
    ap.add_argument("--lr", type=float, default=1e-3)
    ap.add_argument("--mode", choices=["bench", "kernels"], default="bench")
    ap.add_argument("--flush", action="store_true", help="kernels mode: cold Infinity Cache before each FP64 action")
    ap.add_argument("--kernels-elem", choices=["tet4", "hex8"], default="tet4",
                    help="kernels mode: the Tet4 workload (64^3 by default) or a Hex8 compression mesh (--n)")
    args = ap.parse_args()
    if args.gpus != 1:
        print(f"bench.py runs on one GPU only (got --gpus {args.gpus}); the multi-GPU "
              "sharding of this path is a design, not a build.", file=sys.stderr)
        sys.exit(2)

    import torch
    from paper_2602_12365_amd import Operator, inputs as I

    dev = torch.device("cuda", 0)
    torch.cuda.set_device(dev)
    if args.mode == "kernels":
        kernels_mode(args, dev)
        return
    n = args.n
    log(f"mesh n={n}")
    mesh = I.tet_mesh(n)
    ndof = mesh.n_dofs
    u_h = I.gaussian_field(mesh.n_nodes, I.cube_amplitude(n), 0)
    u = torch.as_tensor(u_h).to(dev)
    V = torch.stack([torch.as_tensor(I.unit_direction(mesh.n_nodes, 100 + k)) for k in range(N_DIRS)]).to(dev)
    V32 = V.float()
    Y = torch.empty((mesh.n_nodes, 3), dtype=torch.float64, device=dev)
    Y32 = torch.empty((mesh.n_nodes, 3), dtype=torch.float32, device=dev)

    t0 = time.time()
    op = Operator(I.TET4, mesh.X, mesh.conn, device=dev)
    setup_s = time.time() - t0
    info = op.info()
    log(f"setup {setup_s:.2f}s info={info}")
    stream = torch.cuda.current_stream(dev)

    # events around the 100 tangent actions of every timed step: the
    # dominant kernel's time (chunk pass + halo gather, the launches of
    # efem_hvp) comes from the timed loop itself, so 100 x kernel_us stays
    # below ms_per_step (which adds the linearization)
    hvp_events = []

    def step_f64():
        op.linearize(u, "f64")
        ev = None
        if len(hvp_events) < args.steps:
            ev = (torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True))
            ev[0].record(stream)
        for k in range(N_DIRS):
            op.hvp(V[k], out=Y)
        if ev is not None:
            ev[1].record(stream)
            hvp_events.append(ev)

    for _ in range(args.warmup):
        step_f64()
    torch.cuda.synchronize()
    hvp_events.clear()
    log("warmup done")
    t_step = event_time(step_f64, args.steps, stream)
    value = N_DIRS * ndof / t_step / 1e9
    log(f"f64 step {t_step*1e3:.3f} ms -> {value:.2f} GDoF/s")
    t_acc = sum(a.elapsed_time(b) for a, b in hvp_events) * 1e-3 / (len(hvp_events) * N_DIRS)
    conn_b = mesh.n_elems * 4 * 4
    node_b = mesh.n_nodes * 3 * 8
    alg_hvp, alg_flops = tet4_hvp_alg(mesh.n_elems, mesh.n_nodes, info["n_items"])
    achieved = alg_hvp / t_acc / 1e9
    achieved_tf = alg_flops / t_acc / 1e12
    log(f"hvp chunk pass + gather in the timed steps {t_acc*1e6:.2f} us -> {achieved:.0f} GB/s, "
        f"{achieved_tf:.2f} TFLOP/s")

    # the same launch pair with the 256 MB Infinity Cache flushed before each
    # call (a 512 MiB fill), timed by events around the action alone: the
    # 64^3 working set (~52 MB) otherwise stays cache-resident between calls
    flush = torch.empty(512 << 20, dtype=torch.uint8, device=dev)
    evs = [(torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True))
           for _ in range(40)]
    for ev0, ev1 in evs:
        flush.fill_(1)
        ev0.record(stream)
        op.hvp_zeroed(V[0], Y)
        ev1.record(stream)
    torch.cuda.synchronize()
    t_cold = float(np.median([ev0.elapsed_time(ev1) for ev0, ev1 in evs[5:]])) * 1e-3
    del flush
    log(f"hvp chunk pass + gather, cache flushed: {t_cold*1e6:.2f} us")

    # achievable HBM bandwidth: a plain 1 GiB device copy (read + write)
    ca = torch.empty(1 << 30, dtype=torch.uint8, device=dev)
    cb = torch.empty_like(ca)
    cb.copy_(ca)
    t_copy = event_time(lambda: cb.copy_(ca), 20, stream)
    copy_gbs = 2 * ca.numel() / t_copy / 1e9
    del ca, cb
    log(f"1 GiB device copy: {copy_gbs:.0f} GB/s")

    # FP32 tangent action
    op.linearize(u, "f32")

    def step_f32():
        for k in range(N_DIRS):
            op.hvp(V32[k], out=Y32)
    step_f32()
    t32 = event_time(step_f32, max(args.steps // 2, 2), stream) / N_DIRS
    alg32 = mesh.n_elems * 16 + 4 * mesh.n_nodes * 12

    # energy and residual
    R = torch.empty_like(Y)
    t_res = event_time(lambda: op.residual(u, out=R), 50, stream)
    psi = torch.empty((), dtype=torch.float64, device=dev)
    t_en = event_time(lambda: op.energy(u, out=psi), 50, stream)

    # the other two ways of summing over nodes shared between blocks
    t_scatter, n_col = {}, 0
    for mode in ("color", "atomic"):
        opc = Operator(I.TET4, mesh.X, mesh.conn, scatter=mode, device=dev)
        opc.linearize(u, "f64")
        opc.hvp(V[0], out=Y)
        t_scatter[mode] = event_time(lambda: opc.hvp(V[0], out=Y), 200, stream)
        if mode == "color":
            n_col = opc.info()["n_colours"]
        opc.close()

    # the small-strain linear model on the same mesh (the density of the
    # paper's linear-elastic example): its tangent has no state, so one
    # action reads X and v and writes y
    opl = Operator(I.TET4, mesh.X, mesh.conn, model="linear", device=dev)
    opl.linearize(u, "f64")
    opl.hvp(V[0], out=Y)
    t_l64 = event_time(lambda: opl.hvp(V[0], out=Y), 200, stream)
    opl.linearize(u, "f32")
    opl.hvp(V32[0], out=Y32)
    t_l32 = event_time(lambda: opl.hvp(V32[0], out=Y32), 200, stream)
    t_lres = event_time(lambda: opl.residual(u, out=R), 50, stream)
    t_len = event_time(lambda: opl.energy(u, out=psi), 50, stream)
    opl.close()
    b_l64 = conn_b + 3 * node_b
    b_l32 = conn_b + 3 * node_b // 2
    linear = {
        "hvp_f64_us": round(t_l64 * 1e6, 3), "hvp_f64_gdofs": round(ndof / t_l64 / 1e9, 3),
        "hvp_f64_pct_hbm": round(100 * b_l64 / t_l64 / 1e9 / HBM_PEAK_GBS, 2),
        "hvp_f32_us": round(t_l32 * 1e6, 3), "hvp_f32_gdofs": round(ndof / t_l32 / 1e9, 3),
        "hvp_f32_pct_hbm": round(100 * b_l32 / t_l32 / 1e9 / HBM_PEAK_GBS, 2),
        "residual_us": round(t_lres * 1e6, 3),
        "residual_pct_hbm": round(100 * (conn_b + 3 * node_b) / t_lres / 1e9 / HBM_PEAK_GBS, 2),
        "energy_us": round(t_len * 1e6, 3),
        "energy_pct_hbm": round(100 * (conn_b + 2 * node_b) / t_len / 1e9 / HBM_PEAK_GBS, 2),
        "alg_bytes_hvp_f64": b_l64,
    }
    log(f"linear model: hvp f64 {t_l64*1e6:.2f} us ({linear['hvp_f64_pct_hbm']}% HBM), "
        f"f32 {t_l32*1e6:.2f} us, residual {t_lres*1e6:.2f} us, energy {t_len*1e6:.2f} us")

    # the non-variational transport operator (virtual work): three species,
    # D = 0.1, k = 1/dt = 10, b = omega x x; its tangent action, and one
    # implicit step with the x = 0 face held solved by GMRES(30)
    opt = Operator(I.TET4, mesh.X, mesh.conn, model="transport", device=dev)
    ne_ = mesh.n_elems
    opt.set_material(torch.full((ne_,), 0.1, dtype=torch.float64, device=dev),
                     torch.full((ne_,), 10.0, dtype=torch.float64, device=dev))
    opt.set_velocity([0.6, -1.0, 2.2])
    opt.linearize(u, "f64")
    opt.hvp(V[0], out=Y)
    t_t64 = event_time(lambda: opt.hvp(V[0], out=Y), 200, stream)
    tmask = torch.zeros((mesh.n_nodes, 3), dtype=torch.uint8, device=dev)
    tmask[torch.as_tensor(mesh.X[:, 0] < 1e-12, device=dev)] = 1
    opt.set_dirichlet(tmask)
    zero = torch.zeros_like(u)
    opt.gmres_solve(zero, V[1], rtol=1e-8, restart=30)   # warm-up
    torch.cuda.synchronize()
    t0 = time.time()
    _, gm_it, gm_rr, gm_ok = opt.gmres_solve(zero, V[1], rtol=1e-8, restart=30)
    torch.cuda.synchronize()
    t_gm = time.time() - t0
    opt.close()
    transport = {
        "hvp_f64_us": round(t_t64 * 1e6, 3), "hvp_f64_gdofs": round(ndof / t_t64 / 1e9, 3),
        "hvp_f64_pct_hbm": round(100 * b_l64 / t_t64 / 1e9 / HBM_PEAK_GBS, 2),
        "gmres": {"restart": 30, "rtol": 1e-8, "iterations": gm_it, "relres": gm_rr, "converged": gm_ok,
                  "wall_ms": round(t_gm * 1e3, 3), "ms_per_iteration": round(t_gm * 1e3 / max(gm_it, 1), 4)},
        "case": "D=0.1, k=1/dt=10, omega=(0.6,-1,2.2), x=0 face held, rhs = unit direction seed 101",
    }
    log(f"transport: hvp {t_t64*1e6:.2f} us, gmres {gm_it} its to {gm_rr:.2e} in {t_gm*1e3:.1f} ms")

    # the 2D setup (Tri3, plane strain: out-of-plane components held), the
    # paper's 2D JVP throughput configuration; DOFs counted in plane
    n2 = args.n2d
    m2 = I.tri_mesh(n2)
    dof2 = m2.n_dofs
    op2 = Operator(I.TRI3, m2.X, m2.conn, device=dev)
    op2.set_dirichlet(torch.as_tensor(I.planar_mask(m2.X)).to(dev))
    u2 = torch.as_tensor(I.gaussian_field(m2.n_nodes, 0.01 * 8 / n2, 0)).to(dev)
    u2[:, 2] = 0
    v2 = torch.as_tensor(I.unit_direction(m2.n_nodes, 100)).to(dev)
    y2 = torch.empty_like(v2)
    planar = {"mesh": f"unit square {n2}^2 cells x 2 triangles: {m2.n_elems} Tri3, {m2.n_nodes} nodes, "
                      f"{dof2} in-plane DOF", "paper_context": "matrix-free JVP ~47 MDoF/s in 2D, A100 (JAX)"}
    for model in ("neo_hookean", "linear"):
        op2.set_model(model)
        op2.linearize(u2, "f64")
        op2.hvp(v2, out=y2)
        t2 = event_time(lambda: op2.hvp(v2, out=y2), 200, stream)
        b2 = m2.n_elems * 12 + (4 if model == "neo_hookean" else 3) * m2.n_nodes * 16
        planar[model] = {"hvp_f64_us": round(t2 * 1e6, 3), "hvp_f64_gdofs": round(dof2 / t2 / 1e9, 3),
                         "hvp_f64_pct_hbm_2d_bytes": round(100 * b2 / t2 / 1e9 / HBM_PEAK_GBS, 2)}
        log(f"2D {model}: hvp {t2*1e6:.2f} us -> {dof2 / t2 / 1e9:.2f} GDoF/s")
    op2.close()
    del m2, u2, v2, y2

    # sparse tangent by colouring (Alg. 2): K(u) from n_colours tangent
    # actions, then products by 3x3 blocks against the matrix-free one
    sp_info = op.sparse_setup()
    vals = op.sparse_assemble(u)
    t_asm = event_time(lambda: op.sparse_assemble(u, values=vals), 3, stream)
    t_spmv = event_time(lambda: op.sparse_spmv(vals, V[0], out=Y), 50, stream)
    # what the product by 3x3 blocks moves: every value, one column index
    # per block, the node-row block offsets, x once and y
    spmv_bytes = (sp_info["nnz"] * 8 + sp_info["n_blocks"] * 4 + (sp_info["n_rows"] // 3 + 1) * 8
                  + 2 * ndof * 8)
    sparse = {"n_colours": sp_info["n_colours"], "nnz": sp_info["nnz"],
              "setup_s": round(sp_info["setup_seconds"], 3), "assemble_ms": round(t_asm * 1e3, 3),
              "assemble_gdofs": round(ndof / t_asm / 1e9, 4),
              "spmv_us": round(t_spmv * 1e6, 3), "spmv_gbs": round(spmv_bytes / t_spmv / 1e9, 1),
              "spmv_pct_hbm": round(100 * spmv_bytes / t_spmv / 1e9 / HBM_PEAK_GBS, 2),
              "paper_context": "sparse differentiation ~0.5 MDoF/s in 3D, 80-90 colours, A100 (JAX)"}
    log(f"sparse: {sp_info['n_colours']} colours, nnz {sp_info['nnz']}, assemble {t_asm*1e3:.2f} ms, "
        f"spmv {t_spmv*1e6:.1f} us")
    del vals

    # adjoints on the same mesh with a heterogeneous material (mu lognormal(0,
    # 0.3) seed 4, lam = 1.5): the energy's material and coordinate gradients
    # and the residual's material VJP at u; then the derivative of the top
    # face's total z reaction through the equilibrium solve (bottom clamped,
    # top +0.05 z in 5 steps) by the adjoint method
    from paper_2602_12365_amd import adjoint as A
    mu4 = torch.as_tensor(I.lognormal_field(mesh.n_elems, 0.3, 4)).to(dev)
    opa = Operator(I.TET4, mesh.X, mesh.conn, device=dev)
    opa.set_material(mu4, torch.full_like(mu4, 1.5))
    t_gm = event_time(lambda: opa.grad_material(u), 50, stream)
    t_gx = event_time(lambda: opa.grad_coords(u, out=Y), 50, stream)
    t_vjp = event_time(lambda: opa.residual_vjp_material(u, V[0]), 50, stream)
    mask4, ubc4 = I.clamp_top_bottom(mesh.X, 0.05)
    opa.set_dirichlet(torch.as_tensor(mask4).to(dev))
    ua = torch.zeros_like(u)
    torch.cuda.synchronize()
    t0 = time.time()
    rc_a, st_a = opa.newton_solve(ua, torch.as_tensor(ubc4).to(dev), n_steps=5)
    t_eq = time.time() - t0
    sel = np.zeros((mesh.n_nodes, 3), dtype=np.uint8)
    sel[I.face_nodes(mesh.X, 2, 1.0), 2] = 1
    sel_d = torch.as_tensor(sel.reshape(-1)).to(dev)
    A.reaction_gradient(opa, ua, sel_d)
    torch.cuda.synchronize()
    t0 = time.time()
    _, _, adj_it = A.reaction_gradient(opa, ua, sel_d)
    torch.cuda.synchronize()
    t_adj = time.time() - t0
    adjoints = {
        "material": "mu lognormal(0, 0.3) seed 4, lam 1.5",
        "grad_material_us": round(t_gm * 1e6, 3),
        "grad_coords_us": round(t_gx * 1e6, 3),
        "residual_vjp_material_us": round(t_vjp * 1e6, 3),
        "reaction_gradient": {
            "load_case": "bottom clamped, top +0.05 z in 5 steps; J = total z reaction of the top face",
            "equilibrium_solve_s": round(t_eq, 3), "equilibrium_rc": rc_a,
            "equilibrium_newton_iters": st_a["newton_iters"], "equilibrium_cg_iters": st_a["cg_iters"],
            "adjoint_s": round(t_adj, 4), "adjoint_cg_iters": adj_it,
        },
    }
    log(f"adjoints: grad_material {t_gm*1e6:.1f} us, grad_coords {t_gx*1e6:.1f} us, "
        f"vjp {t_vjp*1e6:.1f} us; reaction gradient {t_adj*1e3:.1f} ms ({adj_it} CG)")
    opa.close()
    del mu4, ua

    hex8 = hex8_section(args, dev, stream)

    t_hvp = t_step / N_DIRS
    # the roofline's bound is the longer of the formulation's two ideal
    # times, alg_bytes / 8 TB/s and alg_flops / 78.6 TFLOP/s; both fractions
    # are reported (hbm_frac is the metric's %HBM)
    if roofline_bound(alg_hvp, alg_flops) == "hbm":
        roof_head = {"bound": "hbm", "achieved": round(achieved, 1), "peak": HBM_PEAK_GBS, "unit": "GB/s",
                     "frac": round(achieved / HBM_PEAK_GBS, 4)}
    else:
        roof_head = {"bound": "alu", "achieved": round(achieved_tf, 3), "peak": FP64_PEAK_TFLOPS,
                     "unit": "TFLOP/s", "frac": round(achieved_tf / FP64_PEAK_TFLOPS, 4)}
    out = {
        "metric": "HVP Gdof/s & %HBM peak; Newton solve s to 1e-8 resid, plain vs mixed+NN",
        "value": round(value, 3),
        "unit": "GDoF/s",
        "n_gpus": 1,
        "steps": args.steps,
        "warmup": args.warmup,
        "ms_per_step": round(t_step * 1e3, 4),
        "higher_is_better": True,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": "f64",
        "data": "synthetic",
        "config": {
            "workload": f"unit cube {n}^3 hexes x 6 Kuhn tets: {mesh.n_elems} Tet4, "
                        f"{mesh.n_nodes} nodes, {ndof} DOF; neo-Hookean mu=1 lam=1.5; "
                        f"u=0.00125*N(0,1); step = linearize + {N_DIRS} FP64 HVPs",
            "scatter": "halo",
            "blocks": info["n_blocks"],
        },
        "roofline": {
            **roof_head,
            "traffic": measured_traffic(),
            "kernel": "k_chunk_hvp64<false, true> + k_halo_gather<double, false, false> (efem_hvp, the "
                      "100 distinct directions of each timed step, events around them)",
            "traffic_note": "L2<->fabric bytes per launch pair from rocprofv3 FETCH_SIZE + WRITE_SIZE, scaled "
                            "by a 256 MiB copy; the same after an Infinity Cache flush",
            "kernel_us": round(t_acc * 1e6, 3),
            "alg_flops": alg_flops,
            "alg_bytes": alg_hvp,
            "hbm_achieved_gbs": round(achieved, 1),
            "hbm_frac": round(achieved / HBM_PEAK_GBS, 4),
            "hbm_copy_gbs": round(copy_gbs, 1),   # achievable: 1 GiB device copy
            "hbm_frac_of_copy": round(achieved / copy_gbs, 4),
            "kernel_us_cache_flushed": round(t_cold * 1e6, 3),
            "hbm_frac_cache_flushed": round(alg_hvp / t_cold / 1e9 / HBM_PEAK_GBS, 4),
            "alu_achieved_tflops": round(achieved_tf, 3),
            "alu_frac": round(achieved_tf / FP64_PEAK_TFLOPS, 4),
        },
        "hvp_f64_us": round(t_hvp * 1e6, 3),
        "hvp_f64_pct_hbm": round(100 * alg_hvp / t_hvp / 1e9 / HBM_PEAK_GBS, 2),
        "hvp_f32_us": round(t32 * 1e6, 3),
        "hvp_f32_gdofs": round(ndof / t32 / 1e9, 3),
        "hvp_f32_pct_hbm": round(100 * alg32 / t32 / 1e9 / HBM_PEAK_GBS, 2),
        "hvp_f64_color_us": round(t_scatter["color"] * 1e6, 3),
        "color_passes": n_col,
        "hvp_f64_atomic_us": round(t_scatter["atomic"] * 1e6, 3),
        "residual_us": round(t_res * 1e6, 3),
        "energy_us": round(t_en * 1e6, 3),
        "setup_s": round(setup_s, 3),
        "adjoints": adjoints,
        "sparse_tangent": sparse,
        "linear_model": linear,
        "transport": transport,
        "planar_2d": planar,
        "hex8": hex8,
        "paper_context": "matrix-free JVP ~13 MDoF/s, 3D linear tets, NVIDIA A100 (JAX), precision unstated",
    }

    if not args.no_solve:
        out["newton"] = solve_section(args, dev)

    if not args.no_cpu:
        from oracle import fem as F
        orc = F.FEM(I.TET4, mesh.X, mesh.conn, np.ones(mesh.n_elems), 1.5 * np.ones(mesh.n_elems))
        v0 = V[0].cpu().numpy()
        orc.hvp(u_h, v0)
        t0 = time.time()
        k = 0
        while k < 3 or time.time() - t0 < args.cpu_seconds:
            orc.hvp(u_h, v0)
            k += 1
        tc = (time.time() - t0) / k
        out["cpu_baseline"] = {
            "value": round(ndof / tc / 1e9, 6),
            "unit": "GDoF/s",
            "cores": F.num_threads(),
            "kind": "oracle",
            "sample": f"{k} full-mesh FP64 tangent actions of the same workload "
                      f"({tc*1e3:.1f} ms each, explicit 81-entry tangent, OpenMP)",
        }
        log(f"oracle {tc*1e3:.1f} ms per HVP on {F.num_threads()} threads")

    op.close()
    print(json.dumps(out), flush=True)


if __name__ == "__main__":
    main()
