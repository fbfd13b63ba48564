"""Benchmark: queries/s at recall@10 = 0.95, FINGER vs plain greedy search on
one MI355X, with the search kernel's achieved HBM bandwidth.

Workload (default): n = 1,000,000 points, m = 128, integer features 0..255
from a 1,000-cluster mixture; graph = exact 16-NN symmetrized and pruned to
degree 32 with reachability repair; 4,096 pivot entry points; FINGER rank
r = 64 with fp32 edge codes; 10,000 queries from the same mixture; K = 10.
All inputs are synthetic and seeded (workloads package).

Flow: build inputs and the exact ground truth (finger_exact_knn), build the
FINGER tables, sweep ef for both modes to find the smallest ef with
recall@10 >= 0.95, then time K steps (one step = query preparation + search
of all queries at that ef) after W warm-up steps.  Prints ONE JSON line on
stdout; progress goes to stderr.

    python bench.py [--gpus 1] [--steps 20] [--warmup 3]
"""
from __future__ import annotations

import argparse
import hashlib
import re
import json
import os
import sys
import time

import numpy as np

ROOT = os.path.dirname(os.path.abspath(__file__))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)

PEAK_HBM_GBS = 8000.0
EF_SWEEP = (10, 12, 16, 20, 24, 28, 32, 36, 40, 44, 48, 52, 56, 60, 64, 72, 80, 96, 112, 128, 160, 200)
TARGET_RECALL = 0.95


def log(*a):
    print("[bench]", *a, file=sys.stderr, flush=True)


def algorithmic_bytes(ctr: np.ndarray, m: int, deg: int, r: int, code_bytes: int,
                      k: int, fp8: bool) -> float:
    """Bytes the method must move for one launch, summed over its queries:
    the query, one adjacency row per expansion, one vector per exact
    distance, c.c and P c per screening expansion, one edge code (plus
    alpha_d, rho_d, and the per-node scale for FP8) per screened edge, and
    the K results."""
    exp, exact, scr, preps = (ctr[:, 0].astype(np.float64), ctr[:, 1].astype(np.float64),
                              ctr[:, 2].astype(np.float64), ctr[:, 5].astype(np.float64))
    per_q = (4 * m + exp * 4 * deg + exact * 4 * m + preps * 4 * (r + 1)
             + scr * (r * code_bytes + 8) + (preps * 4 if fp8 else 0) + 8 * k)
    return float(per_q.sum())


def kernel_source_hash() -> str:
    """Hash of the search kernel's code: comments, trailing blanks and blank
    lines are dropped, so that editing a comment keeps counters taken on the
    same code valid."""
    h = hashlib.sha256()
    for f in ("search_kernel.h", "search_rule.h", "search.hip", "device_common.h"):
        with open(os.path.join(ROOT, "paper_2206_11408_amd", "csrc", f)) as fh:
            text = fh.read()
        text = re.sub(r"/\*.*?\*/", " ", text, flags=re.S)
        text = re.sub(r"//[^\n]*", "", text)
        h.update("\n".join(ln.rstrip() for ln in text.splitlines() if ln.strip()).encode())
    return h.hexdigest()[:16]


def measured_traffic(mode_name: str, workload: str):
    """HBM bytes per launch from the committed rocprofv3 counter summary, if it
    was taken on the current search kernel source; else None."""
    path = os.path.join(ROOT, "profiles", "search_c2_counters.json")
    try:
        with open(path) as f:
            rec = json.load(f)
    except (OSError, ValueError):
        return None
    if rec.get("kernel_source_hash") != kernel_source_hash() or rec.get("workload") != workload:
        return None
    ent = rec.get("modes", {}).get(mode_name)
    return None if ent is None else ent.get("hbm_bytes_per_launch")


def c4_leg(a, log, tune_mod) -> dict:
    """The batching workload (DEEP-10M-96's shape): n points from a mixture
    of 10,000 Gaussians in 96-d (sigma 0.5), graph = 16-NN symmetrized and
    pruned to degree 32 with repair, built with each point's kNN taken
    within its own mixture component (finger_build_graph_grouped; the
    exactness of that shortcut is measured on a sample), FINGER tables at
    r = 32 with FP8 edge codes, 16,384 pivot entry points, and 100,000
    queries with K drawn from {1, 10, 100} and ef from {32, ..., 512}.  One
    step = query preparation + one search call over all queries: the ef-class
    partition (one persistent launch per class) against a single launch that
    reserves LDS for ef_max in every wave, FINGER and plain."""
    import torch
    from paper_2206_11408_amd import _lib as L
    from paper_2206_11408_amd import api
    from workloads import SPECS, make_points, pick_pivots
    dev = torch.device("cuda")
    spec = SPECS["c4"]
    if a.c4_n != spec.n:
        spec = spec.scaled(n=a.c4_n, n_centers=max(10, spec.n_centers * a.c4_n // spec.n))
    t0 = time.time()
    data, queries, lab = make_points(spec, labels=True)
    order = np.argsort(lab, kind="stable")
    data = np.ascontiguousarray(data[order])
    offs = np.concatenate([[0], np.cumsum(np.bincount(lab, minlength=spec.n_centers))]).astype(np.int64)
    del lab, order
    log(f"c4: {spec.n} x {spec.m} points (sorted by component) and {spec.nq} queries in {time.time() - t0:.1f}s")
    d_data = torch.as_tensor(data, device=dev)
    d_q = torch.as_tensor(queries, device=dev)
    torch.cuda.synchronize()
    t0 = time.time()
    dG, gst = api.finger_build_graph_grouped(d_data, offs, knn_k=spec.knn_k, max_degree=spec.max_degree,
                                             entry=0)
    torch.cuda.synchronize()
    graph_s = time.time() - t0
    log(f"c4: grouped graph in {graph_s:.1f}s: {gst}")
    # the grouped kNN is the exact kNN for a point whose knn_k + 1 nearest
    # (itself included) all lie in its own component: checked on a sample
    rng = np.random.default_rng(11)
    samp = np.sort(rng.choice(spec.n, 2000, replace=False))
    si, _ = api.finger_exact_knn(d_data, d_data[torch.as_tensor(samp, device=dev)], spec.knn_k + 1)
    comp = np.searchsorted(offs, np.arange(spec.n), side="right") - 1
    si = si.cpu().numpy()
    grouped_exact = float(np.mean([(comp[si[i]] == comp[samp[i]]).all() for i in range(samp.size)]))
    log(f"c4: sampled points whose exact {spec.knn_k}-NN lie in their own component: {grouped_exact:.4f}")
    t0 = time.time()
    piv = pick_pivots(spec.n, 16384, spec.seed)
    tab = api.finger_build_tables(d_data, dG, rank=32, code_type=L.CODE_FP8E4M3, pivots=piv, seed=0)
    torch.cuda.synchronize()
    tables_s = time.time() - t0
    log(f"c4: FINGER tables r=32 fp8 in {tables_s:.1f}s")
    nq = spec.nq
    qrng = np.random.default_rng(4)
    K = qrng.choice([1, 10, 100], size=nq).astype(np.int32)
    EF = qrng.choice([32, 64, 128, 256, 512], size=nq).astype(np.int32)
    dK, dEF = torch.as_tensor(K, device=dev), torch.as_tensor(EF, device=dev)
    t0 = time.time()
    gi, _ = api.finger_exact_knn(d_data, d_q, 100)
    gi = gi.cpu().numpy()
    log(f"c4: exact 100-NN of {nq} queries in {time.time() - t0:.1f}s")

    def recall(ids):
        return float(np.mean([np.isin(ids[i, :K[i]], gi[i, :K[i]]).sum() / K[i] for i in range(nq)]))

    out = {"workload": (f"c4: n={spec.n} m={spec.m} float32, {spec.n_centers}-component Gaussian mixture "
                        f"(sigma {spec.sigma}), 16-NN within components sym pruned deg 32, 16384 pivots, "
                        f"r=32 fp8 codes, nq={nq}, K in {{1,10,100}}, ef in {{32,...,512}} per query"),
           "graph_s": round(graph_s, 2), "tables_s": round(tables_s, 2),
           "components_before_repair": gst["components_before_repair"],
           "grouped_knn_exact_fraction": round(grouped_exact, 4)}
    ev0, ev1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    kev = (torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True))
    for e in kev:   # create the HIP events (torch records them once) before they are handed over
        e.record()
    for name, mode, cls in (("finger", L.MODE_FINGER, 0), ("finger_classes", L.MODE_FINGER, 1),
                            ("finger_single_reservation", L.MODE_FINGER, 2), ("plain", L.MODE_PLAIN, 0),
                            ("plain_classes", L.MODE_PLAIN, 1)):
        base = dict(mode=mode, k=100, k_max=100, ef=32, entry=-1, k_per_query=dK, ef_per_query=dEF,
                    ef_max=512, persistent=1, ef_classes=cls)
        geo = {}
        if a.tune:
            ch = tune_mod.autotune(tab, d_q, base, repeats=2, cache_path=None)
            geo = {k: ch[k] for k in ("waves_per_cu", "code_prefetch", "visited_capacity", "visited_probe")}
        p = api.search_params(**{**base, **geo})
        outb = (torch.empty((nq, 100), dtype=torch.int32, device=dev),
                torch.empty((nq, 100), dtype=torch.float32, device=dev),
                torch.empty((nq, L.NCOUNTERS), dtype=torch.int32, device=dev))
        for _ in range(max(1, a.warmup)):
            api.finger_search(tab, d_q, p, out=outb, check=False)
        torch.cuda.synchronize()
        steps = max(3, a.steps // 4)
        kms = []
        ev0.record()
        for _ in range(steps):
            p.kernel_events[0] = kev[0].cuda_event
            p.kernel_events[1] = kev[1].cuda_event
            api.finger_search(tab, d_q, p, out=outb, check=False)
        ev1.record()
        torch.cuda.synchronize()
        ms = ev0.elapsed_time(ev1) / steps
        kms = kev[0].elapsed_time(kev[1])   # the last step's search launches
        api.check_status(outb[2])
        ids, ctr = outb[0].cpu().numpy(), outb[2].cpu().numpy()
        B = algorithmic_bytes(ctr, spec.m, spec.max_degree, 32 if mode else 0, 1, 100, True)
        out[name] = dict(qps=round(nq / ms * 1e3, 1), ms_per_step=round(ms, 3), search_ms=round(kms, 3),
                         recall=round(recall(ids), 4), alg_gbs=round(B / (kms * 1e-3) / 1e9, 1),
                         hbm_frac=round(B / (kms * 1e-3) / 1e9 / PEAK_HBM_GBS, 4),
                         exact=round(float(ctr[:, 1].mean()), 1), screened=round(float(ctr[:, 2].mean()), 1),
                         skipped=round(float(ctr[:, 3].mean()), 1), launch=geo or "library default")
        log(f"c4 {name}: {out[name]}")
    # the default (one launch, largest ef class first) against one launch per
    # class and against one launch serving the queries in index order
    out["longest_first_vs_classes"] = round(out["finger"]["qps"] / out["finger_classes"]["qps"], 4)
    out["longest_first_vs_query_order"] = round(out["finger"]["qps"] / out["finger_single_reservation"]["qps"], 4)
    out["finger_vs_plain"] = round(out["finger"]["qps"] / out["plain"]["qps"], 4)
    if a.cpu_sample > 0:
        # the float64 oracle (compiled) on a sample of one (K, ef) group
        from oracle import csearch
        from oracle.build import build as oracle_build
        t0 = time.time()
        G = dG.cpu().numpy()
        orc = oracle_build(data, G, 32, n_samples=100_000, seed=0)
        sel = np.nonzero((K == 10) & (EF == 64))[0][: max(64, a.cpu_sample // 8)]
        from oracle.search import pivot_entries
        ent = pivot_entries(queries[sel], data, piv)
        X64 = data.astype(np.float64)
        cores = max(1, min(16, len(os.sched_getaffinity(0))))
        w0 = time.perf_counter()
        csearch.search_batch(X64, G, queries[sel].astype(np.float64), ent, 64, 10, mode="finger",
                             tables=orc, threads=cores)
        out["cpu_oracle"] = {"qps": round(sel.size / (time.perf_counter() - w0), 2), "cores": cores,
                             "sample": f"{sel.size} queries with K=10, ef=64, FINGER mode, float64 basis "
                                       f"(not the fp8 codes)"}
        del X64
        log(f"c4 oracle: {out['cpu_oracle']} (setup {time.time() - t0:.1f}s)")
    tab.close()
    del d_data, d_q, dG
    torch.cuda.empty_cache()
    return out


def main() -> int:
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=20)
    ap.add_argument("--warmup", type=int, default=3)
    ap.add_argument("--n", type=int, default=1_000_000)
    ap.add_argument("--clusters", type=int, default=1000)
    ap.add_argument("--nq", type=int, default=10_000)
    ap.add_argument("--rank", type=int, default=64)
    ap.add_argument("--code", choices=("f32", "bf16", "fp8"), default="f32")
    ap.add_argument("--pivots", type=int, default=4096)
    ap.add_argument("--cpu-sample", type=int, default=4000,
                    help="queries of the oracle CPU baseline (0 = skip)")
    ap.add_argument("--extra-codes", default="",
                    help="comma list of extra FINGER variants to sweep and report: "
                         "code[:pf|:nopf] with code in f32,bf16,fp8 (pf = edge codes requested "
                         "with the adjacency row)")
    ap.add_argument("--ef-plain", type=int, default=0, help="skip the plain sweep, use this ef")
    ap.add_argument("--ef-finger", type=int, default=0, help="skip the FINGER sweep, use this ef")
    ap.add_argument("--gate", type=int, default=5000,
                    help="train the learned gate on this many extra queries (0 = skip) and "
                         "report the gated search (cascade and every edge) at matched recall")
    ap.add_argument("--gate-band", type=float, default=0.25,
                    help="cascade band: the gate decides edges within band * ub^2 of the bound")
    ap.add_argument("--ablation", action="store_true",
                    help="also run the ablation variants (low-rank only, random projections with "
                         "and without distribution matching) and the rank rule")
    ap.add_argument("--no-tune", dest="tune", action="store_false",
                    help="time the default launch geometry instead of the autotuned one")
    ap.add_argument("--hierarchy", action="store_true",
                    help="also build HNSW-style upper layers (M = 16) and report both modes "
                         "started from the descent instead of the nearest pivot")
    ap.add_argument("--spectrum", action=argparse.BooleanOptionalAction, default=True,
                    help="also report plain and FINGER (r = 64 and r = 16) on the same recipe with a "
                         "decaying noise spectrum calibrated to the paper's SIFT rank")
    ap.add_argument("--spectrum-codes", default="",
                    help="extra FINGER code variants (code[:pf|:nopf]) on the spectrum leg")
    ap.add_argument("--wide", default="c3s,c3b",
                    help="comma-separated precision workloads: 1M x 960 (c3a: isotropic noise, c3s: decaying "
                         "spectrum) on which to also measure plain and FINGER (bf16 and fp8 codes); "
                         "empty to skip")
    ap.add_argument("--wide-rule-rank", action="store_true",
                    help="on the 960-d workloads also measure FINGER at r = 16 (the rank rule's choice)")
    ap.add_argument("--mips", action="store_true",
                    help="also report both modes under the inner-product metric (FINGER_IP) on the "
                         "same points and graph, against inner-product ground truth")
    ap.add_argument("--oracle-legs", type=int, default=0,
                    help="time the float64 oracle on this many queries for the --mips and "
                         "--hierarchy legs (0 = skip)")
    ap.add_argument("--graph", action=argparse.BooleanOptionalAction, default=False,
                    help="time the step as a replay of a captured HIP graph (kernel times "
                         "still come from the eager launches)")
    ap.add_argument("--c4", action=argparse.BooleanOptionalAction, default=True,
                    help="the batching leg: 10M x 96, r=32 fp8, 100k queries with mixed K/ef")
    ap.add_argument("--c4-n", type=int, default=10_000_000, help="points of the batching leg")
    ap.add_argument("--screen-layout", type=int, default=0, choices=(0, 1, 2),
                    help="FINGER screen: 0 library default, 1 coalesced, 2 per-lane chunks")
    ap.add_argument("--copy-probe", action="store_true",
                    help="also run one 1 GiB device copy (the reference kernel for HBM counters)")
    a = ap.parse_args()

    if a.gpus != 1 or int(os.environ.get("WORLD_SIZE", "1")) != 1:
        print("bench.py measures one GPU only: it runs the per-shard search on a "
              "single MI355X; the index would be sharded by queries or by data across GPUs, "
              "which is not run here. Use --gpus 1.",
              file=sys.stderr)
        return 2

    import torch
    from paper_2206_11408_amd import _lib as L
    from paper_2206_11408_amd import api, tune
    from workloads import SPECS, make_points, medoid, pick_pivots

    if not torch.cuda.is_available():
        print("bench.py needs a GPU", file=sys.stderr)
        return 2
    dev = torch.device("cuda:0")
    code_of = {"f32": (L.CODE_F32, 4), "bf16": (L.CODE_BF16, 2), "fp8": (L.CODE_FP8E4M3, 1)}

    # ------------------------------------------------------------ inputs
    spec = SPECS["c2"].scaled(n=a.n, n_centers=a.clusters, nq=a.nq)
    t0 = time.time()
    data, queries = make_points(spec)
    log(f"points n={a.n} m={spec.m} nq={a.nq} in {time.time() - t0:.1f}s")
    d_data = torch.as_tensor(data, device=dev)
    d_q = torch.as_tensor(queries, device=dev)
    d_q_main = d_q
    t0 = time.time()
    d_G, gstats = api.finger_build_graph(d_data, knn_k=spec.knn_k, max_degree=spec.max_degree,
                                         entry=medoid(data))
    torch.cuda.synchronize()
    graph_s = time.time() - t0
    log(f"graph (on the GPU) in {graph_s:.2f}s: {gstats}")
    G = d_G.cpu().numpy()
    piv = pick_pivots(a.n, a.pivots, spec.seed)
    t0 = time.time()
    gt_ids, gt_d = api.finger_exact_knn(d_data, d_q, 10)
    torch.cuda.synchronize()
    log(f"ground truth (exact kNN, MFMA) in {time.time() - t0:.2f}s")
    gt_ids = gt_ids.cpu().numpy()
    gt_d = gt_d.cpu().numpy()

    def recall(ids, dist, gt=None):
        # tie-aware: a returned id also counts if it sits at the 10th distance
        g_ids, g_d = gt if gt is not None else (gt_ids, gt_d)
        kth = g_d[:, 9:10]
        hit = (ids[:, :10, None] == g_ids[:, None, :10]).any(2) | ((dist[:, :10] <= kth) & (ids[:, :10] >= 0))
        return float(hit.mean())

    tables = {}

    def get_tables(code):
        if code not in tables:
            t0 = time.time()
            tables[code] = api.finger_build_tables(d_data, d_G, rank=a.rank, code_type=code_of[code][0],
                                                   pivots=piv, seed=0)
            torch.cuda.synchronize()
            inf = tables[code].info()
            log(f"FINGER tables r={a.rank} {code} in {time.time() - t0:.1f}s: mu={inf['mu']:.4f} "
                f"sigma={inf['sigma']:.4f} mu_hat={inf['mu_hat']:.4f} sigma_hat={inf['sigma_hat']:.4f} "
                f"eps={inf['eps']:.4f} edge bytes={inf['edge_table_bytes'] / 1e9:.2f} GB")
        return tables[code]

    ev = (torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True))
    kev = (torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True))
    for e in ev + kev:   # torch creates the HIP event on first record
        e.record()
    torch.cuda.synchronize()

    launch = {}   # (mode, code) -> tuned launch settings

    def run(tab, mode, ef, out=None, time_kernel=False, prefetch=0, entry=L.ENTRY_PIVOT, queries=None,
            band=0.0):
        p = api.search_params(mode=mode, k=10, ef=ef, entry=entry, code_prefetch=prefetch,
                              screen_layout=a.screen_layout, gate_band=band)
        if time_kernel:
            p.kernel_events[0] = kev[0].cuda_event
            p.kernel_events[1] = kev[1].cuda_event
        return api.finger_search(tab, d_q if queries is None else queries, p, out=out, check=False)

    def sweep(tab, mode, prefetch=0, entry=L.ENTRY_PIVOT, gt=None, queries=None, efs=EF_SWEEP, band=0.0):
        res = []
        for ef in efs:
            run(tab, mode, ef, prefetch=prefetch, entry=entry, queries=queries, band=band)
            torch.cuda.synchronize()
            ev[0].record()
            ids, dist, ctr = run(tab, mode, ef, prefetch=prefetch, entry=entry, queries=queries, band=band)
            ev[1].record()
            torch.cuda.synchronize()
            ms = ev[0].elapsed_time(ev[1])
            rc = recall(ids.cpu().numpy(), dist.cpu().numpy(), gt)
            api.check_status(ctr)
            c = ctr.cpu().numpy()
            res.append(dict(ef=ef, recall=rc, ms=ms, qps=a.nq / ms * 1e3,
                            exact=float(c[:, 1].mean()), screened=float(c[:, 2].mean()),
                            skipped=float(c[:, 3].mean()), expansions=float(c[:, 0].mean()),
                            status_bad=int((c[:, 6] != 0).sum())))
            log(f"  mode={mode} ef={ef:4d} recall={rc:.4f} {ms:7.3f} ms  qps={a.nq / ms * 1e3:,.0f} "
                f"exp={res[-1]['expansions']:.1f} exact={res[-1]['exact']:.1f} "
                f"scr={res[-1]['screened']:.1f} skip={res[-1]['skipped']:.1f}")
            if rc >= TARGET_RECALL + 0.01 and ef >= 16:
                break
        ok = [r for r in res if r["recall"] >= TARGET_RECALL]
        return res, (min(ok, key=lambda r: r["ef"]) if ok else max(res, key=lambda r: r["recall"]))

    def timed(tab, mode, ef, steps, warmup, code_bytes, fp8, prefetch=0, entry=L.ENTRY_PIVOT, gt=None,
              queries=None, rank=None, m=None, band=0.0):
        nq = a.nq
        d_q = d_q_main if queries is None else queries
        out = (torch.empty((nq, 10), dtype=torch.int32, device=dev),
               torch.empty((nq, 10), dtype=torch.float32, device=dev),
               torch.empty((nq, L.NCOUNTERS), dtype=torch.int32, device=dev))
        if a.tune:
            base = dict(mode=mode, k=10, ef=ef, entry=entry, screen_layout=a.screen_layout, gate_band=band)
            ch = tune.autotune(tab, d_q, base, repeats=3, cache_path=None, log=log)
            if prefetch != 0:   # an explicitly requested code-prefetch setting stays fixed
                best = min((t, c) for t, c in ch["all"] if c["code_prefetch"] == prefetch)[1]
                ch = dict(best)
            launch[(mode, id(tab), prefetch, entry)] = {k: ch[k] for k in
                                                        ("waves_per_cu", "persistent", "code_prefetch",
                                                         "visited_capacity", "visited_probe")}
            log(f"tuned launch mode={mode}: {launch[(mode, id(tab), prefetch, entry)]}")
        geo = launch.get((mode, id(tab), prefetch, entry), {})
        p = api.search_params(mode=mode, k=10, ef=ef, entry=entry, screen_layout=a.screen_layout, gate_band=band,
                              code_prefetch=geo.get("code_prefetch", prefetch),
                              waves_per_cu=geo.get("waves_per_cu", 0),
                              persistent=geo.get("persistent", 0),
                              visited_capacity=geo.get("visited_capacity", 0),
                              visited_probe=geo.get("visited_probe", 0))
        for _ in range(warmup):
            api.finger_search(tab, d_q, p, out=out, check=False)
        pairs = [(torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True))
                 for _ in range(steps)]
        for e0, e1 in pairs:   # create the HIP events before the timed region
            e0.record()
            e1.record()
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        ev[0].record()
        for e0, e1 in pairs:
            p.kernel_events[0] = e0.cuda_event
            p.kernel_events[1] = e1.cuda_event
            api.finger_search(tab, d_q, p, out=out, check=False)
        ev[1].record()
        torch.cuda.synchronize()
        total = time.perf_counter() - t0
        gpu_total = ev[0].elapsed_time(ev[1]) * 1e-3
        kms = [e0.elapsed_time(e1) for e0, e1 in pairs]
        graph_step = None
        if a.graph:
            # the same step captured once in a HIP graph and replayed: query
            # preparation and search without per-launch host gaps
            pg = api.search_params(mode=mode, k=10, ef=ef, entry=entry, screen_layout=a.screen_layout, gate_band=band,
                                   code_prefetch=geo.get("code_prefetch", prefetch),
                                   waves_per_cu=geo.get("waves_per_cu", 0),
                                   persistent=geo.get("persistent", 0),
                                   visited_capacity=geo.get("visited_capacity", 0),
                              visited_probe=geo.get("visited_probe", 0))
            side = torch.cuda.Stream()
            side.wait_stream(torch.cuda.current_stream())
            with torch.cuda.stream(side):
                api.finger_search(tab, d_q, pg, out=out, check=False)
            torch.cuda.current_stream().wait_stream(side)
            torch.cuda.synchronize()
            cg = torch.cuda.CUDAGraph()
            with torch.cuda.graph(cg):
                api.finger_search(tab, d_q, pg, out=out, check=False)
            for _ in range(warmup):
                cg.replay()
            torch.cuda.synchronize()
            g0 = time.perf_counter()
            for _ in range(steps):
                cg.replay()
            torch.cuda.synchronize()
            graph_step = (time.perf_counter() - g0) / steps
            del cg
        api.check_status(out[2])   # after the timed region: no visited-set overflow
        ids, dist, ctr = (x.cpu().numpy() for x in out)
        B = algorithmic_bytes(ctr, spec.m if m is None else m, spec.max_degree, (a.rank if rank is None else rank) if mode else 0,
                              code_bytes, 10, fp8)
        kavg = float(np.mean(kms))
        if graph_step is not None:
            log(f"  graph replay: {graph_step * 1e3:.4f} ms per step (eager {total / steps * 1e3:.4f})")
            total = graph_step * steps
        return dict(ef=ef, launch=geo, qps=nq * steps / total, ms_per_step=total / steps * 1e3,
                    graph=graph_step is not None,
                    gpu_ms_per_step=gpu_total / steps * 1e3,
                    kernel_ms=kavg, kernel_ms_min=float(np.min(kms)), alg_bytes=B,
                    alg_gbs=B / (kavg * 1e-3) / 1e9, recall=recall(ids, dist, gt),
                    exact=float(ctr[:, 1].mean()), skipped=float(ctr[:, 3].mean()),
                    screened=float(ctr[:, 2].mean()))

    tabF = get_tables(a.code)
    if a.copy_probe:
        src = torch.empty(1 << 30, dtype=torch.uint8, device=dev)
        dst = torch.empty_like(src)
        dst.copy_(src)
        torch.cuda.synchronize()
        del src, dst
        log("copy probe: 1 GiB device-to-device copy done")
    if a.ef_plain:
        op_p = {"ef": a.ef_plain, "recall": float("nan")}
    else:
        log("sweep plain")
        sw_p, op_p = sweep(tabF, L.MODE_PLAIN)
    if a.ef_finger:
        op_f = {"ef": a.ef_finger, "recall": float("nan")}
    else:
        log("sweep finger")
        sw_f, op_f = sweep(tabF, L.MODE_FINGER)
    log(f"operating points: plain ef={op_p['ef']} recall={op_p['recall']:.4f}; "
        f"finger ef={op_f['ef']} recall={op_f['recall']:.4f}")

    cb, fp8 = code_of[a.code][1], a.code == "fp8"
    # timed region: plain baseline, then FINGER (the metric)
    tp = timed(tabF, L.MODE_PLAIN, op_p["ef"], a.steps, a.warmup, cb, fp8)
    log(f"plain  timed: {tp}")
    tf = timed(tabF, L.MODE_FINGER, op_f["ef"], a.steps, a.warmup, cb, fp8)
    log(f"finger timed: {tf}")

    extra = {}
    for variant in [c for c in a.extra_codes.split(",") if c]:
        code, _, pfs = variant.partition(":")
        pf = {"pf": 1, "nopf": -1, "": 0}[pfs]
        tab = get_tables(code)
        if a.ef_finger:   # a fixed FINGER operating point applies to every code variant
            op = {"ef": a.ef_finger}
        else:
            sw, op = sweep(tab, L.MODE_FINGER, prefetch=pf)
        tx = timed(tab, L.MODE_FINGER, op["ef"], a.steps, a.warmup, code_of[code][1], code == "fp8",
                   prefetch=pf)
        extra[variant] = dict(ef=op["ef"], recall=round(tx["recall"], 4), qps=round(tx["qps"], 1),
                              kernel_ms=round(tx["kernel_ms"], 4), alg_gbs=round(tx["alg_gbs"], 1),
                              launch=tx["launch"],
                              speedup_vs_plain=round(tx["qps"] / tp["qps"], 4))
        log(f"finger {variant} timed: {tx}")

    def oracle_qps(fn, count):
        """The float64 oracle on `count` queries, one thread: queries/s."""
        from threadpoolctl import threadpool_limits
        with threadpool_limits(limits=1):
            w0 = time.perf_counter()
            fn(count)
            return round(count / (time.perf_counter() - w0), 2)

    mips = None
    if a.mips:
        from oracle.search import pivot_entries as o_piv, search_batch as o_search
        tabI = api.finger_build_tables(d_data, d_G, rank=a.rank, metric=L.IP, pivots=piv, seed=0)
        gi, gd = api.finger_exact_knn(d_data, d_q, 10, metric=L.IP)
        gtI = (gi.cpu().numpy(), gd.cpu().numpy())
        mips = {}
        for nm, mode in (("plain", L.MODE_PLAIN), ("finger", L.MODE_FINGER)):
            log(f"sweep {nm}, inner product")
            sw, op = sweep(tabI, mode, gt=gtI)
            th = timed(tabI, mode, op["ef"], a.steps, a.warmup, cb, fp8, gt=gtI)
            log(f"{nm} timed, inner product: {th}")
            mips[nm] = dict(ef=op["ef"], recall=round(th["recall"], 4), qps=round(th["qps"], 1),
                            kernel_ms=round(th["kernel_ms"], 4), exact=round(th["exact"], 1),
                            alg_gbs=round(th["alg_gbs"], 1), launch=th["launch"])
        mips["speedup_vs_plain"] = round(mips["finger"]["qps"] / mips["plain"]["qps"], 4)
        if a.oracle_legs:
            from oracle.build import build as oracle_build
            orc_t = oracle_build(data, G, a.rank, n_samples=100_000, seed=0)
            qs_o = queries[:a.oracle_legs]
            mips["oracle_qps_finger"] = oracle_qps(
                lambda c: o_search(data, G, qs_o[:c], o_piv(qs_o[:c], data, piv, metric="ip"),
                                   mips["finger"]["ef"], 10, mode="finger", tables=orc_t, metric="ip"),
                a.oracle_legs)
        tabI.close()

    sift = None
    if a.spectrum:
        # the same recipe with a decaying noise spectrum (the rank rule settles
        # on r = 16 there, as the paper reports for SIFT-1M-128): plain,
        # FINGER at the configured rank and FINGER at the rule's rank
        spec2 = SPECS["c2s"].scaled(n=a.n, n_centers=a.clusters, nq=a.nq)
        data2, q2 = make_points(spec2)
        dd2 = torch.as_tensor(data2, device=dev)
        dq2 = torch.as_tensor(q2, device=dev)
        t0 = time.time()
        dG2, gst2 = api.finger_build_graph(dd2, knn_k=spec2.knn_k, max_degree=spec2.max_degree,
                                           entry=medoid(data2))
        torch.cuda.synchronize()
        log(f"c2s graph in {time.time() - t0:.1f}s: {gst2}")
        piv2 = pick_pivots(a.n, a.pivots, spec2.seed)
        gi2, gd2 = api.finger_exact_knn(dd2, dq2, 10)
        gt2 = (gi2.cpu().numpy(), gd2.cpu().numpy())
        t64 = api.finger_build_tables(dd2, dG2, rank=a.rank, pivots=piv2, seed=0)
        t16 = api.finger_build_tables(dd2, dG2, rank=16, pivots=piv2, seed=0)
        sift = {"workload": (f"c2s: n={a.n} m=128 int 0-255, {a.clusters}-cluster mixture with noise "
                             f"spectrum i^-{spec2.decay}, 16-NN sym pruned deg 32, {a.pivots} pivots, "
                             f"nq={a.nq}, K=10"),
                "corr_xy_r16": round(t16.info()["corr_xy"], 4),
                "corr_xy_r64": round(t64.info()["corr_xy"], 4)}
        for nm, tab, mode, r in (("plain", t64, L.MODE_PLAIN, 0), ("finger_r64", t64, L.MODE_FINGER, a.rank),
                                 ("finger_r16", t16, L.MODE_FINGER, 16)):
            log(f"sweep {nm} (c2s)")
            sw, op = sweep(tab, mode, gt=gt2, queries=dq2)
            th = timed(tab, mode, op["ef"], a.steps, a.warmup, 4, False, gt=gt2, queries=dq2, rank=r)
            log(f"{nm} timed (c2s): {th}")
            sift[nm] = dict(ef=op["ef"], recall=round(th["recall"], 4), qps=round(th["qps"], 1),
                            kernel_ms=round(th["kernel_ms"], 4), exact=round(th["exact"], 1),
                            screened=round(th["screened"], 1), skipped=round(th["skipped"], 1),
                            alg_gbs=round(th["alg_gbs"], 1),
                            hbm_frac=round(th["alg_gbs"] / PEAK_HBM_GBS, 4), launch=th["launch"])
        for variant in [c for c in a.spectrum_codes.split(",") if c]:
            code, _, pfs = variant.partition(":")
            pf = {"pf": 1, "nopf": -1, "": 0}[pfs]
            tv = api.finger_build_tables(dd2, dG2, rank=a.rank, code_type=code_of[code][0], pivots=piv2,
                                         seed=0)
            sw, op = sweep(tv, L.MODE_FINGER, prefetch=pf, gt=gt2, queries=dq2)
            th = timed(tv, L.MODE_FINGER, op["ef"], a.steps, a.warmup, code_of[code][1], code == "fp8",
                       prefetch=pf, gt=gt2, queries=dq2, rank=a.rank)
            log(f"finger {variant} timed (c2s): {th}")
            sift[f"finger_r64_{variant}"] = dict(
                ef=op["ef"], recall=round(th["recall"], 4), qps=round(th["qps"], 1),
                kernel_ms=round(th["kernel_ms"], 4), exact=round(th["exact"], 1),
                alg_gbs=round(th["alg_gbs"], 1), launch=th["launch"],
                speedup_vs_plain=round(th["qps"] / sift["plain"]["qps"], 4))
            tv.close()
        sift["speedup_r64_vs_plain"] = round(sift["finger_r64"]["qps"] / sift["plain"]["qps"], 4)
        sift["speedup_r16_vs_plain"] = round(sift["finger_r16"]["qps"] / sift["plain"]["qps"], 4)
        t64.close()
        t16.close()
        del dd2, dq2, dG2

    wide = {}
    angular = {}
    for wname in [w for w in a.wide.split(",") if w]:
        # a 960-d workload (GIST-1M-960's shape): a vector is 3,840 bytes
        # against 136 (bf16) or 72 (fp8) bytes per edge code at r = 64, the
        # regime where screening can pay in bytes if the residuals are low-rank;
        # c3b (GloVe-1.2M-100's shape): 100-d heavy-tailed vectors under the
        # angular metric (Supplementary A), every row scaled by a random
        # factor so that the metric's normalization matters
        spec3 = SPECS[wname].scaled(nq=a.nq)
        ang = wname == "c3b"
        metric3 = L.ANGULAR if ang else L.L2
        t0 = time.time()
        data3, q3 = make_points(spec3)
        if ang:
            srng = np.random.default_rng(3)
            data3 = (data3 * srng.uniform(0.5, 4.0, (data3.shape[0], 1))).astype(np.float32)
            q3 = (q3 * srng.uniform(0.5, 4.0, (q3.shape[0], 1))).astype(np.float32)
        dd3 = torch.as_tensor(data3, device=dev)
        dq3 = torch.as_tensor(q3, device=dev)
        log(f"{wname} points n={spec3.n} m={spec3.m} in {time.time() - t0:.1f}s")
        t0 = time.time()
        ent3 = medoid(data3 / np.linalg.norm(data3, axis=1, keepdims=True) if ang else data3)
        dG3, gst3 = api.finger_build_graph(dd3, knn_k=spec3.knn_k, max_degree=spec3.max_degree,
                                           entry=ent3, metric=metric3)
        torch.cuda.synchronize()
        log(f"{wname} graph in {time.time() - t0:.1f}s: {gst3}")
        piv3 = pick_pivots(spec3.n, a.pivots, spec3.seed)
        gi3, gd3 = api.finger_exact_knn(dd3, dq3, 10, metric=metric3)
        gt3 = (gi3.cpu().numpy(), gd3.cpu().numpy())
        if ang:
            desc = (f"{wname}: n={spec3.n} m={spec3.m} float32, {spec3.n_centers} N(0,I) centres + Student-t(3) "
                    f"noise, rows scaled by U(0.5, 4), angular metric, 16-NN sym pruned deg 32, {a.pivots} "
                    f"pivots, nq={a.nq}, K=10")
        else:
            noise = f"noise spectrum i^-{spec3.decay}" if spec3.decay > 0 else "isotropic noise"
            desc = (f"{wname}: n={spec3.n} m={spec3.m} float32, {spec3.n_centers} uniform centres + "
                    f"{spec3.sigma} Gaussian {noise}, 16-NN sym pruned deg 32, {a.pivots} pivots, "
                    f"nq={a.nq}, K=10")
        res = {"workload": desc}
        efs3 = EF_SWEEP + (256, 320, 400)
        for rank in (a.rank, 16) if a.wide_rule_rank and a.rank != 16 else (a.rank,):
            for code in ("bf16", "fp8"):
                tw = api.finger_build_tables(dd3, dG3, rank=rank, code_type=code_of[code][0], pivots=piv3,
                                             seed=0, metric=metric3)
                res[f"corr_xy_r{rank}"] = round(tw.info()["corr_xy"], 4)
                legs = [(f"finger_{code}_r{rank}", L.MODE_FINGER)]
                if code == "bf16" and rank == a.rank:
                    legs.insert(0, ("plain", L.MODE_PLAIN))   # plain reads no codes
                for nm, mode in legs:
                    log(f"sweep {nm} ({wname})")
                    sw, op = sweep(tw, mode, gt=gt3, queries=dq3, efs=efs3)
                    th = timed(tw, mode, op["ef"], a.steps, a.warmup, code_of[code][1], code == "fp8",
                               gt=gt3, queries=dq3, rank=rank, m=spec3.m)
                    log(f"{nm} timed ({wname}): {th}")
                    res[nm] = dict(ef=op["ef"], recall=round(th["recall"], 4), qps=round(th["qps"], 1),
                                   kernel_ms=round(th["kernel_ms"], 4), exact=round(th["exact"], 1),
                                   screened=round(th["screened"], 1), skipped=round(th["skipped"], 1),
                                   alg_gbs=round(th["alg_gbs"], 1),
                                   hbm_frac=round(th["alg_gbs"] / PEAK_HBM_GBS, 4), launch=th["launch"])
                    if mode == L.MODE_FINGER:
                        res[nm]["speedup_vs_plain"] = round(th["qps"] / res["plain"]["qps"], 4)
                tw.close()
        (angular if ang else wide)[wname] = res
        del dd3, dq3, dG3
        torch.cuda.empty_cache()

    hier = None
    if a.hierarchy:
        from workloads import build_hierarchy, draw_levels
        t0 = time.time()
        levels = draw_levels(a.n, 16, spec.seed)
        upper, top = build_hierarchy(data, levels, M=16, device="cuda")
        api.finger_hierarchy_attach(tabF, levels, upper)
        log(f"hierarchy M=16 in {time.time() - t0:.1f}s: top level {levels.max()}, "
            f"{upper.shape[0]} upper rows, top node {top}")
        api.finger_descend(tabF, d_q)
        torch.cuda.synchronize()
        ev[0].record()
        for _ in range(a.steps):
            dent, dcalls = api.finger_descend(tabF, d_q)
        ev[1].record()
        torch.cuda.synchronize()
        d_ms = ev[0].elapsed_time(ev[1]) / a.steps
        hier = {"levels": int(levels.max()), "upper_rows": int(upper.shape[0]),
                "descent_ms": round(d_ms, 4), "descent_calls": round(float(dcalls.float().mean()), 1)}
        for nm, mode in (("plain", L.MODE_PLAIN), ("finger", L.MODE_FINGER)):
            log(f"sweep {nm} from descent entries")
            sw, op = sweep(tabF, mode, entry=L.ENTRY_DESCENT)
            th = timed(tabF, mode, op["ef"], a.steps, a.warmup, cb, fp8, entry=L.ENTRY_DESCENT)
            log(f"{nm} timed from descent entries: {th}")
            hier[nm] = dict(ef=op["ef"], recall=round(th["recall"], 4), qps=round(th["qps"], 1),
                            kernel_ms=round(th["kernel_ms"], 4), exact=round(th["exact"], 1),
                            launch=th["launch"])
        hier["speedup_vs_plain"] = round(hier["finger"]["qps"] / hier["plain"]["qps"], 4)
        if a.oracle_legs:
            from oracle.search import hierarchy_entries
            qs_o = queries[:a.oracle_legs]
            hier["oracle_descent_qps"] = oracle_qps(
                lambda c: hierarchy_entries(qs_o[:c], data, levels, upper), a.oracle_legs)
        hier["pivot_entries"] = dict(plain_exact=round(tp["exact"], 1), finger_exact=round(tf["exact"], 1))

    gated = None
    if a.gate > 0:
        from paper_2206_11408_amd import gate as gate_mod
        tr_spec = SPECS["c2"].scaled(n=a.n, n_centers=a.clusters, nq=a.nq + a.gate)
        _, tr_q = make_points(tr_spec)   # same mixture; rows after the first nq are new draws
        t0 = time.time()
        info = gate_mod.fit_gate(tabF, torch.as_tensor(tr_q[a.nq:], device=dev), ef=op_f["ef"],
                                 hidden=64, epochs=2, batch=4096, lr=2e-3,
                                 capacity=min(20_000_000, max(1 << 20, 1000 * a.gate)),
                                 log=log)
        torch.cuda.synchronize()
        log(f"gate trained in {time.time() - t0:.1f}s on {info['rows']} rows "
            f"(screened {info['screened']}), loss {info['loss']}, eps_gate {info['eps_gate']:.4f}")
        gated = dict(train_queries=a.gate, train_rows=info["rows"], eps_gate=round(info["eps_gate"], 5),
                     train_s=round(time.time() - t0, 2), loss=[round(x, 5) for x in info["loss"]])
        for nm, band in (("cascade", a.gate_band), ("every_edge", 0.0)):
            sw_g, op_g = sweep(tabF, L.MODE_GATED, band=band)
            tg = timed(tabF, L.MODE_GATED, op_g["ef"], a.steps, a.warmup, cb, fp8, band=band)
            log(f"gated ({nm}) timed: {tg}")
            gated[nm] = dict(band=band, ef=op_g["ef"], recall=round(tg["recall"], 4), qps=round(tg["qps"], 1),
                             kernel_ms=round(tg["kernel_ms"], 4), exact=round(tg["exact"], 1),
                             skipped=round(tg["skipped"], 1), speedup_vs_plain=round(tg["qps"] / tp["qps"], 4),
                             speedup_vs_finger=round(tg["qps"] / tf["qps"], 4))
        gated["finger"] = dict(ef=op_f["ef"], exact=round(tf["exact"], 1), skipped=round(tf["skipped"], 1))

    ablation_out = None
    if a.ablation:
        from paper_2206_11408_amd import ablation
        from workloads import gaussian_projection
        proj = gaussian_projection(a.rank, spec.m, 7)
        ablation_out = {}
        nq_err = min(2000, a.nq)
        for v in ablation.VARIANTS:
            tab = tabF if v == "finger" else ablation.variant_tables(
                d_data, d_G, a.rank, v, projection=proj, pivots=piv, seed=0)
            sw, op = sweep(tab, L.MODE_FINGER)
            err = ablation.approximation_error(tab, d_q[:nq_err], op["ef"])
            curve = [dict(ef=r_["ef"], recall=round(r_["recall"], 4),
                          effective_calls=round(r_["exact"] + r_["screened"] * a.rank / spec.m, 1),
                          exact=round(r_["exact"], 1), ms=round(r_["ms"], 3)) for r_ in sw]
            ablation_out[v] = dict(ef=op["ef"], recall=round(op["recall"], 4), qps=round(op["qps"], 1),
                                   effective_calls=round(op["exact"] + op["screened"] * a.rank / spec.m, 1),
                                   approx_error_median=round(err["median"], 5),
                                   approx_error_p90=round(err["p90"], 5), curve=curve)
            log(f"ablation {v}: {ablation_out[v] | {'curve': len(curve)}}")
            if v != "finger":
                tab.close()
        r_sel, t_sel, hist = ablation.select_rank(d_data, d_G, target=0.7, pivots=piv, seed=0)
        sw, op = sweep(t_sel, L.MODE_FINGER)
        ablation_out["rank_rule"] = dict(rank=r_sel, corr_history=[(r_, round(c_, 4)) for r_, c_ in hist],
                                         ef=op["ef"], recall=round(op["recall"], 4),
                                         qps=round(op["qps"], 1),
                                         effective_calls=round(op["exact"] + op["screened"] * r_sel / spec.m, 1))
        ablation_out["plain"] = dict(ef=op_p["ef"], effective_calls=round(tp["exact"], 1))
        log(f"rank rule: {ablation_out['rank_rule']}")
        t_sel.close()

    # ------------------------------------------------------ CPU baseline
    cpu = None
    if a.cpu_sample > 0:
        from oracle.build import build as oracle_build
        from oracle.search import pivot_entries, search_batch
        t0 = time.time()
        orc = oracle_build(data, G, a.rank, n_samples=100_000, seed=0)
        log(f"oracle tables in {time.time() - t0:.1f}s")
        qs = queries[:a.cpu_sample]
        from threadpoolctl import threadpool_limits
        with threadpool_limits(limits=1):   # the oracle is single-threaded; keep BLAS so too
            w0 = time.perf_counter()
            ent = pivot_entries(qs, data, piv)
            py_ids = search_batch(data, G, qs, ent, op_f["ef"], 10, mode="finger", tables=orc)[0]
            wall = time.perf_counter() - w0
        numpy_qps = a.cpu_sample / wall
        # the compiled float64 search on every host core (independent threads
        # over disjoint query ranges), and on one of them
        from oracle import csearch
        X64 = np.ascontiguousarray(data, dtype=np.float64)
        Q64 = np.ascontiguousarray(qs, dtype=np.float64)
        # the GPU machine allots a share of 16 host cores to its one GPU (more
        # threads would compete with the other tenants of the host), so the
        # oracle runs on min(16, affinity) threads; the counts and the CPU
        # model are recorded with the result
        affinity = len(os.sched_getaffinity(0))
        cores = max(1, min(16, affinity))
        cpu_model = "unknown"
        try:
            with open("/proc/cpuinfo") as f:
                cpu_model = next((ln.split(":", 1)[1].strip() for ln in f if ln.startswith("model name")),
                                 "unknown")
        except OSError:
            pass
        n1 = min(a.cpu_sample, 1000)
        w0 = time.perf_counter()
        c1 = csearch.search_batch(X64, G, Q64[:n1], ent[:n1], op_f["ef"], 10, mode="finger", tables=orc)
        c_single = n1 / (time.perf_counter() - w0)
        w0 = time.perf_counter()
        csearch.search_batch(X64, G, Q64, ent, op_f["ef"], 10, mode="finger", tables=orc, threads=cores)
        c_all = a.cpu_sample / (time.perf_counter() - w0)
        del X64
        cpu = {"value": round(c_all, 3), "unit": "queries/s", "cores": cores, "kind": "oracle",
               "sample": f"{a.cpu_sample} of the {a.nq} queries, FINGER mode at ef={op_f['ef']}, "
                         f"compiled float64 oracle search on {cores} threads over disjoint query "
                         f"ranges (entries and tables precomputed)",
               "cpu_model": cpu_model, "os_cpu_count": os.cpu_count(), "affinity_cpus": affinity,
               "cores_policy": "min(16, affinity): the GPU box's host share for one GPU",
               "single_thread_qps": round(c_single, 3),
               "numpy_oracle_one_core_qps": round(numpy_qps, 3),
               "numpy_oracle_sample": f"{a.cpu_sample} queries, entry selection included",
               # two renderings of the same search: identical top-K expected
               "oracles_agree": round(float((c1[0] == py_ids[:n1]).all(1).mean()), 4)}
        log(f"cpu oracle: {cpu}")

    workload = (f"c2: n={a.n} m={spec.m} int 0-255, {a.clusters}-cluster mixture, 16-NN sym pruned "
                f"deg 32, {a.pivots} pivots, r={a.rank} {a.code} codes, nq={a.nq}, K=10")
    traffic = measured_traffic("finger", workload)
    # what a plain streaming kernel reaches on this GPU, beside the published
    # peak: STREAM's scale (b = 1.0 * a) over 4 GiB of float32, 4 GiB read
    # and 4 GiB written (well past the last-level cache), best of 10, timed
    # with events on the stream it runs on.  (torch's same-dtype copy_ takes
    # the runtime's blit path, which measured about 13% slower.)
    src = torch.ones(1 << 30, dtype=torch.float32, device=dev)
    dst = torch.empty_like(src)
    torch.mul(src, 1.0, out=dst)
    best = float("inf")
    for _ in range(10):
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        e0.record()
        torch.mul(src, 1.0, out=dst)
        e1.record()
        e1.synchronize()
        best = min(best, e0.elapsed_time(e1))
    stream_gbs = 2 * (4 << 30) / (best * 1e-3) / 1e9
    del src, dst
    torch.cuda.empty_cache()
    log(f"stream probe: {stream_gbs:.0f} GB/s (scale over 4 GiB, best of 10)")
    roof = {"bound": "hbm", "achieved": round(tf["alg_gbs"], 1), "peak": PEAK_HBM_GBS,
            "unit": "GB/s", "frac": round(tf["alg_gbs"] / PEAK_HBM_GBS, 4),
            "traffic": traffic, "kernel": "k_search (FINGER mode)",
            "kernel_ms": round(tf["kernel_ms"], 4), "alg_bytes_per_launch": round(tf["alg_bytes"]),
            "stream_probe_gbs": round(stream_gbs, 1),
            "frac_of_stream_probe": round(tf["alg_gbs"] / stream_gbs, 4)}
    line = {
        "metric": "queries/sec at recall@10=0.95 (FINGER search, 1 MI355X)",
        "value": round(tf["qps"], 1),
        "unit": "queries/s",
        "n_gpus": 1,
        "steps": a.steps,
        "warmup": a.warmup,
        "ms_per_step": round(tf["ms_per_step"], 4),
        "higher_is_better": True,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": "f32",
        "data": "synthetic",
        "config": {"workload": workload, "ef_finger": op_f["ef"], "ef_plain": op_p["ef"],
                   "recall_finger": round(tf["recall"], 4), "recall_plain": round(tp["recall"], 4),
                   "launch_finger": tf["launch"], "launch_plain": tp["launch"]},
        "plain_qps": round(tp["qps"], 1),
        "speedup_vs_plain": round(tf["qps"] / tp["qps"], 4),
        "plain_roofline": {"achieved": round(tp["alg_gbs"], 1), "frac": round(tp["alg_gbs"] / PEAK_HBM_GBS, 4),
                           "kernel_ms": round(tp["kernel_ms"], 4),
                           "frac_of_stream_probe": round(tp["alg_gbs"] / stream_gbs, 4)},
        "roofline": roof,
        "cpu_baseline": cpu,
    }
    if extra:
        line["extra_codes"] = extra
    if gated:
        line["gated"] = gated
    if ablation_out:
        line["ablation"] = ablation_out
    if hier:
        line["descent_entries"] = hier
    if mips:
        line["inner_product"] = mips
    if sift:
        line["sift_like_spectrum"] = sift
    if wide:
        line["wide_960"] = wide
    if angular:
        line["angular_100"] = angular
    if a.c4:
        line["batching_c4"] = c4_leg(a, log, tune)
    if a.oracle_legs:
        # graph construction at a size the float64 oracle finishes: the first
        # 20,000 points, same recipe, GPU and oracle side by side
        from oracle import graph as o_graph
        sub = np.ascontiguousarray(data[:20_000])
        e_sub = medoid(sub)
        torch.cuda.synchronize()
        t0 = time.time()
        api.finger_build_graph(torch.as_tensor(sub, device=dev), knn_k=spec.knn_k,
                               max_degree=spec.max_degree, entry=e_sub)
        torch.cuda.synchronize()
        g_small = time.time() - t0
        from threadpoolctl import threadpool_limits
        with threadpool_limits(limits=1):
            t0 = time.time()
            o_graph.build(sub, spec.knn_k, spec.max_degree, e_sub)
            o_small = time.time() - t0
        gstats["n20000_gpu_s"] = round(g_small, 3)
        gstats["n20000_oracle_s"] = round(o_small, 2)
    exact_bf16 = bool((d_data == d_data.bfloat16().float()).all())
    line["graph_build"] = {"seconds": round(graph_s, 3), "knn_ms": round(gstats["ms_knn"], 1),
                           "symmetrize_ms": round(gstats["ms_symmetrize"], 1),
                           "prune_ms": round(gstats["ms_prune"], 1), "repair_ms": round(gstats["ms_repair"], 1),
                           # 2 n^2 m useful flops; the split-bf16 scores execute three
                           # products on the matrix cores, or one where every point is
                           # a bf16 value (integers up to 256)
                           "knn_useful_tflops": round(2.0 * a.n * a.n * spec.m / (gstats["ms_knn"] * 1e-3) / 1e12, 1),
                           "knn_bf16_mfma_tflops": round((1 if exact_bf16 else 3) * 2.0 * a.n * a.n * spec.m / (gstats["ms_knn"] * 1e-3) / 1e12, 1)}
    for key in ("n20000_gpu_s", "n20000_oracle_s"):
        if key in gstats:
            line["graph_build"][key] = gstats[key]
    print(json.dumps(line), flush=True)
    return 0


if __name__ == "__main__":
    sys.exit(main())
