"""The work this package is timed on: frames through the estimator, windows
through the two learned scorers, training steps and a serving round, each
through the public entry points a program calls.

A case is a dict of plain values; ``kind`` names the entry point:

  estimate   Estimator.estimate_area (or a captured graph of it) on a batch
  logits     Estimator.cnn_window_logits / cnn2d_window_logits
  train      one training step: cnn_gradients + cnn_sgd_step (or the 2-D pair)
  serve      a Server: one frame of every stream submitted, all of them served
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2210_14771_amd import api, serve, synth, synth_gpu, train_scorer

FRAME_STREAM = 140       # seed stream of the frames drawn here
DEVICE = "cuda:0"


# ------------------------------------------------------------- the cases --

def _estimate(name, w, h, n, hs, vs, attempts, scorer=0, fallback=0.0, form="batch", graph=False):
    """form: "batch" one [n, h, w, 3] tensor; "crops" a list of views into
    larger frames (odd row strides and offsets); "mixed" a list of frames in
    the uneven batch's four resolutions (w, h unused)."""
    c = {"kind": "estimate", "w": w, "h": h, "n": n, "hs": hs, "vs": vs, "attempts": attempts,
         "scorer": scorer, "fallback": fallback, "form": form, "graph": graph}
    return {"name": name, **c} if name else c


def _windows(name, kind, net, frames, strips):
    c = {"kind": kind, "net": net, "frames": frames, "strips": strips}
    return {"name": name, **c} if name else c


def listed():
    return [
        # the least a program asks: one SD frame of a live picture, Table A1's defaults
        _estimate("frame_480p", 640, 480, 1, 16, 16, 256),
        # the small workload: eight SD frames at the defaults
        _estimate("batch_480p", 640, 480, 8, 16, 16, 256),
        # frames cropped out of a capture card's buffer: odd sizes, odd strip
        # counts, unaligned rows, a list of views
        _estimate("crops_odd", 853, 479, 6, 17, 15, 512, form="crops"),
        # the headline workload: 64 full-HD frames, 32 + 32 strips, 1024 attempts
        _estimate("batch_1080p", 1920, 1080, 64, 32, 32, 1024),
        # the uneven batch (SD, HD, full HD and 4K together) replayed from a graph
        _estimate("mixed_graph", 0, 0, 128, 32, 32, 1024, form="mixed", graph=True),
        # the learned scorers with the handcrafted fallback on the headline batch
        _estimate("learned_1080p", 1920, 1080, 64, 32, 32, 1024, 1, 0.5),
        _estimate("learned2d_1080p", 1920, 1080, 64, 32, 32, 1024, 2, 0.5),
        # scoring the windows of a set of frames: judging a model while it is made
        _windows("logits_1d", "logits", "1d", 16, 16),
        _windows("logits_2d", "logits", "2d", 16, 16),
        # the training program's own step: 64 frames, 16 strips of each
        _windows("train_1d", "train", "1d", 64, 16),
        _windows("train_2d", "train", "2d", 64, 16),
        # 48 streams of mixed resolution, one frame of each arriving together
        {"name": "serve_48", "kind": "serve", "streams": 48, "hs": 32, "vs": 32, "attempts": 1024,
         "scorer": 0, "fallback": 0.0, "lend": False},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    pick = rng.random()
    if pick < 0.60:
        scorer = rng.choice([0, 0, 0, 1, 2])
        hs = rng.choice([8, 16, 17, 32, 48])
        vs = rng.choice([0, 8, 15, 16, 32])
        attempts = rng.choice([64, 200, 256, 512, 1024])
        fallback = rng.choice([0.0, 0.5]) if scorer else 0.0
        if rng.random() < 0.15:
            return _estimate(None, 0, 0, rng.randint(8, 96), hs, vs, attempts, scorer, fallback,
                             "mixed", rng.random() < 0.5)
        w = _log_int(rng, 256, 3840)
        h = max(144, min(2160, int(w * rng.uniform(0.5, 0.85))))
        most = max(1, min(64, 64 * 1920 * 1080 // (w * h)))
        n = min(most, _log_int(rng, 1, 64))
        form = rng.choice(["batch", "batch", "crops"])
        return _estimate(None, w, h, n, hs, vs, attempts, scorer, fallback, form,
                         rng.random() < 0.25)
    if pick < 0.72:
        return _windows(None, "logits", rng.choice(["1d", "2d"]), _log_int(rng, 1, 32),
                        _log_int(rng, 1, 16))
    if pick < 0.90:
        return _windows(None, "train", rng.choice(["1d", "2d"]), _log_int(rng, 1, 64),
                        _log_int(rng, 1, 16))
    scorer = rng.choice([0, 0, 1, 2])
    return {"kind": "serve", "streams": _log_int(rng, 1, 48), "hs": rng.choice([16, 32]),
            "vs": rng.choice([16, 32]), "attempts": rng.choice([256, 1024]), "scorer": scorer,
            "fallback": 0.5 if scorer else 0.0, "lend": rng.random() < 0.5}


# ---------------------------------------------------------------- inputs --

def _recipes(shapes, seed):
    """Frames of the headline distribution at the given (w, h)."""
    return [synth_gpu.draw_recipe(synth.HD_1080p, FRAME_STREAM, seed * 1024 + i, False, w, h)
            for i, (w, h) in enumerate(shapes)]


def _shapes(case):
    if case["form"] == "mixed":
        return synth.mixed_shapes(case["n"])
    return [(case["w"], case["h"])] * case["n"]


CROP_X, CROP_Y, CROP_PAD_W, CROP_PAD_H = 5, 3, 12, 7   # of a crop inside its larger frame


def _frames(case, seed):
    shapes = _shapes(case)
    if case["form"] == "crops":
        w, h = case["w"], case["h"]
        big = [(w + CROP_PAD_W, h + CROP_PAD_H)] * case["n"]
        full = synth_gpu.DeviceRecipes(_recipes(big, seed)).render_frames()
        return [f[CROP_Y:CROP_Y + h, CROP_X:CROP_X + w] for f in full]
    flat = synth_gpu.DeviceRecipes(_recipes(shapes, seed)).render_frames()
    if case["form"] == "batch":
        return flat
    if flat.dim() == 4:      # every frame of one size
        return list(flat)
    out, at = [], 0
    for w, h in shapes:
        out.append(flat[at:at + 3 * w * h].view(h, w, 3))
        at += 3 * w * h
    return out


def _params(case):
    return api.default_params(n_hstrips=case["hs"], n_vstrips=case["vs"],
                              ransac_attempts=case["attempts"], scorer=case["scorer"],
                              fallback_inlier_frac=case["fallback"])


def _estimator(scorer):
    est = api.Estimator(DEVICE)
    if scorer == 1:
        est.set_model(train_scorer.load_model())
    elif scorer == 2:
        est.set_model_2d(train_scorer.load_model_2d())
    return est


def _window_batch(case, seed):
    """Windows as the training program draws them: (recipes, descriptors)."""
    rng = np.random.default_rng([seed, 7])
    recs = train_scorer.draw_frames(synth_gpu.TRAIN_PLAIN, synth_gpu.TRAIN_HARD, seed * 64,
                                    case["frames"], 0.5, rng)
    desc = []
    for f, rc in enumerate(recs):    # rows and columns in turn
        w, h = rc.spec.width, rc.spec.height
        for k in range(case["strips"]):
            row = k % 2 == 0
            line = int(rng.integers(0, h if row else w))
            desc.append(synth_gpu.strip_windows(f, row, line, w if row else h))
    return recs, np.concatenate(desc)


def _window_count(case):
    """18 windows a row of a 1080p frame, 10 a column."""
    return case["frames"] * ((case["strips"] + 1) // 2 * 18 + case["strips"] // 2 * 10)


def _window_model(case):
    """A finished scorer to score with; a training run's first weights to train."""
    if case["kind"] == "logits":
        return (train_scorer.load_model_2d() if case["net"] == "2d"
                else train_scorer.load_model())
    if case["net"] == "1d":
        return train_scorer.init_params(0)
    stats = train_scorer.load_model_2d()[:6].astype(np.float64)
    return train_scorer.init_params_2d(0, stats[:3], 1.0 / stats[3:])


def _streams(case, seed):
    """One device frame per stream, the serving shapes in turn."""
    rng = np.random.default_rng([seed, 9])
    out = []
    for sid in range(case["streams"]):
        w, h = serve.SERVE_SHAPES[sid % len(serve.SERVE_SHAPES)]
        recs = serve.drifting_recipes(seed * 64 + sid, w, h, 1, rng)
        out.append(synth_gpu.DeviceRecipes(recs).render_frames()[0])
    return out


def prepare(case, seed):
    kind = case["kind"]
    if kind == "estimate":
        s = {"kind": kind, "est": _estimator(case["scorer"]), "frames": _frames(case, seed),
             "params": _params(case), "graph": None}
        if case["graph"]:
            s["graph"] = s["est"].capture(s["frames"], s["params"])
        return s
    if kind == "serve":
        est = _estimator(case["scorer"])
        cfg = serve.server_config(max_batch=64, n_hstrips=case["hs"], n_vstrips=case["vs"],
                                  ransac_attempts=case["attempts"], scorer=case["scorer"],
                                  fallback_inlier_frac=case["fallback"])
        frames = _streams(case, seed)
        srv = serve.Server(est, cfg)
        for sid, f in enumerate(frames):
            srv.open(sid, f.shape[1], f.shape[0])
        torch.cuda.synchronize()    # the server reads the frames on a stream of its own
        return {"kind": kind, "srv": srv, "frames": frames, "lend": case["lend"], "seq": 0}
    est = _estimator(0)
    (est.set_model_2d if case["net"] == "2d" else est.set_model)(_window_model(case))
    recs, desc = _window_batch(case, seed)
    batch = train_scorer.Batch(recs, desc, 0.0, case["net"])
    return {"kind": kind, "net": case["net"], "est": est, "batch": batch}


# ------------------------------------------------------------------ runs --

def run(s):
    kind = s["kind"]
    if kind == "estimate":
        raw = (s["graph"].launch() if s["graph"] is not None
               else s["est"].estimate_area(s["frames"], s["params"])).raw
        # (cx, cy, r, score) and (inliers, n_points, valid, reason) of every frame
        return {"circle": raw[:, :4].view(torch.float32), "counts": raw[:, 4:]}
    if kind == "serve":
        srv, seq, frames = s["srv"], s["seq"], s["frames"]
        s["seq"] += 1
        for sid, f in enumerate(frames):
            srv.submit(sid, seq, f, s["lend"])
        got = []
        while len(got) < len(frames):
            got += [serve.served_record(r) for r in srv.step()]
        got.sort(key=lambda r: r["stream"])
        return {"circle": np.array([r["result"][:4] for r in got], dtype=np.float32),
                "counts": np.array([r["result"][4:] for r in got], dtype=np.int32),
                "filtered": np.array([r["filtered"][1:] for r in got], dtype=np.float32)}
    est, b = s["est"], s["batch"]
    if kind == "logits":
        if s["net"] == "2d":
            return {"logits": est.cnn2d_window_logits(b.win, b.geom, b.rng)}
        return {"logits": est.cnn_window_logits(b.win, b.rng)}
    # a rate of the ends of the schedule (warm-up, cosine)
    if s["net"] == "2d":
        grad, loss = est.cnn2d_gradients(*b.tensors(), b.scale)
        est.cnn2d_sgd_step(grad, 1e-4, 0.9)
    else:
        grad, loss = est.cnn_gradients(*b.tensors(), b.scale)
        est.cnn_sgd_step(grad, 1e-4, 0.9)
    return {"grad": grad, "loss": loss}


# ------------------------------------------------------------------ work --

def _estimate_work(shapes, case):
    hs, vs, scorer = case["hs"], case["vs"], case["scorer"]
    lines = (3, 8, 7)[scorer]
    per_position = (0, 24352, 19792)[scorer]
    positions = sum(hs * w + vs * h for w, h in shapes)
    # about half of the candidates are kept and tested in each of the three
    # refits and the final pass
    points = hs + vs
    ransac = len(shapes) * case["attempts"] * points * (23 * 3 + 9)
    return {"bytes": positions * lines * 3 + 32 * len(shapes),
            "flops": positions * per_position + ransac}


def work(case):
    if case["kind"] == "estimate":
        return _estimate_work(_shapes(case), case)
    if case["kind"] == "serve":
        shapes = [serve.SERVE_SHAPES[i % len(serve.SERVE_SHAPES)] for i in range(case["streams"])]
        w = _estimate_work(shapes, case)
        if not case["lend"]:    # a submitted frame is copied into its stream's ring
            w["bytes"] += 2 * sum(3 * a * b for a, b in shapes)
        return w
    n = _window_count(case)
    flops = 112 * (24352 if case["net"] == "1d" else 19792)
    bytes_ = 8 * 128 * 3 + 8 + (32 if case["net"] == "2d" else 0)
    if case["kind"] == "logits":
        return {"bytes": n * (bytes_ + 112 * 4), "flops": n * flops}
    return {"bytes": n * (bytes_ + 112 * 8), "flops": 3 * n * flops}


# ----------------------------------------------------------------- exact --
#
# The estimator in numpy: integer luma, Sobel, quantised magnitude and angle,
# float32 score tables, the best pixel of each half strip, then RANSAC in
# 64 bits.  The candidates are integers by definition; the circles are
# 64-bit numbers.

def _lines(frame, pos, horizontal):
    """Luma [strips, 3, length] of the lines pos - 1 .. pos + 1."""
    idx = (pos[:, None] + np.arange(-1, 2)[None, :]).ravel()
    px = (frame[idx] if horizontal else frame[:, idx].transpose(1, 0, 2)).astype(np.int64)
    y = (77 * px[..., 0] + 150 * px[..., 1] + 29 * px[..., 2] + 128) >> 8
    return y.reshape(len(pos), 3, -1)


def _positions(extent, n):
    if n == 0:
        return np.zeros(0, np.int64)
    t = (8.0 / n) * (np.arange(n) - (n - 1) / 2.0)
    return np.clip(np.floor(extent / (1.0 + np.exp(-t))).astype(np.int64), 1, extent - 2)


def _score_tables():
    p = api.default_params()
    q = np.arange(12000)
    sg = np.tanh(q / (8.0 * p.t_g)).astype(np.float32)
    u = np.arange(2049) / 1024.0
    th = np.where(u <= 1.0, np.arctan2(u, 1.0 - u), np.pi - np.arctan2(2.0 - u, u - 1.0))
    st = (1.0 - np.tanh(th * (180.0 / np.pi) / p.t_theta_deg)).astype(np.float32)
    si = (1.0 - np.tanh(np.arange(256) / p.t_iota)).astype(np.float32)
    return sg, st, si


def _candidates(frame, hs, vs, tables):
    """(x, y, score) of the best pixel of every half strip, strips in order."""
    sg, st, si = tables
    H, W, _ = frame.shape
    X, Y, S = [], [], []
    for horizontal, n, extent in ((True, hs, H), (False, vs, W)):
        if n == 0:
            continue
        pos = _positions(extent, n)
        t = _lines(frame, pos, horizontal)
        L = t.shape[2]
        pad = np.pad(t, ((0, 0), (0, 0), (1, 1)), mode="edge")
        s = pad[:, 0] + 2 * pad[:, 1] + pad[:, 2]
        d = pad[:, 2] - pad[:, 0]
        along = s[:, 2:] - s[:, :-2]
        across = d[:, :-2] + 2 * d[:, 1:-1] + d[:, 2:]
        i = np.arange(L)[None, :]
        gx, gy = (along, across) if horizontal else (across, along)
        x, y = (i, pos[:, None]) if horizontal else (pos[:, None], i)
        m2 = gx * gx + gy * gy
        root = np.floor(np.sqrt(64.0 * m2)).astype(np.int64)
        root -= root * root > 64 * m2
        root += (root + 1) * (root + 1) <= 64 * m2
        c2x, c2y = W - 1 - 2 * x, H - 1 - 2 * y
        dt = gx * c2x + gy * c2y
        cr = np.abs(gx * c2y - gy * c2x)
        den = cr + np.abs(dt)
        safe = np.maximum(den, 1)
        f, up = (1024 * cr) // safe, -((-1024 * cr) // safe)
        qt = np.where(den == 0, 0, np.where(dt >= 0, f, 2048 - up))
        part = np.where(m2 == 0, np.float32(0), sg[np.minimum(root, len(sg) - 1)] * st[qt])
        cut = L // 2
        at, best = [], []
        for p, lum, sign in ((part[:, :cut], t[:, 1, :cut], 1),
                             (part[:, cut:][:, ::-1], t[:, 1, cut:][:, ::-1], -1)):
            run_max = np.maximum.accumulate(lum, axis=1)
            iota = np.concatenate([np.zeros((n, 1), np.int64), run_max[:, :-1]], axis=1)
            sc = p * si[iota]
            k = np.argmax(sc, axis=1)
            at.append(k if sign > 0 else L - 1 - k)
            best.append(sc[np.arange(n), k])
        # strip by strip, first half then second
        along_, line = np.stack(at, axis=1).ravel(), np.repeat(pos, 2)
        X.append(along_ if horizontal else line)
        Y.append(line if horizontal else along_)
        S.append(np.stack(best, axis=1).ravel())
    return np.concatenate(X), np.concatenate(Y), np.concatenate(S).astype(np.float32)


def _mulhi(a, b):
    m = np.uint64(0xFFFFFFFF)
    s = np.uint64(32)
    a0, a1, b0, b1 = a & m, a >> s, b & m, b >> s
    p00, p01, p10, p11 = a0 * b0, a0 * b1, a1 * b0, a1 * b1
    mid = (p00 >> s) + (p01 & m) + (p10 & m)
    return p11 + (p01 >> s) + (p10 >> s) + (mid >> s)


def _philox(attempts, uid):
    """Philox4x64-10 (Salmon et al., 2011), key (0, 0), counter (attempt, uid, 0, 0)."""
    with np.errstate(over="ignore"):
        c0 = np.arange(attempts, dtype=np.uint64)
        c1 = np.full(attempts, uid, np.uint64)
        c2, c3 = np.zeros(attempts, np.uint64), np.zeros(attempts, np.uint64)
        k0, k1 = np.uint64(0), np.uint64(0)
        m0, m1 = np.uint64(0xD2E7470EE14C6C93), np.uint64(0xCA5A826395121157)
        for r in range(10):
            if r:
                k0 = k0 + np.uint64(0x9E3779B97F4A7C15)
                k1 = k1 + np.uint64(0xBB67AE8584CAA73B)
            h0, l0, h1, l1 = _mulhi(m0, c0), m0 * c0, _mulhi(m1, c2), m1 * c2
            c0, c1, c2, c3 = h1 ^ c1 ^ k0, l1, h0 ^ c3 ^ k1, l0
    return c0, c1, c2


def _circle(cand, W, H, attempts, uid):
    """(cx, cy, r, score) of one frame, 64-bit, as the method defines it."""
    p = api.default_params()
    x, y, sc = cand
    edge = np.minimum(np.minimum(x, y), np.minimum(W - 1 - x, H - 1 - y))
    keep = (edge >= p.t_px) & (sc >= np.float32(p.t_ps))
    u, v, q = x[keep] - W // 2, y[keep] - H // 2, np.floor(sc[keep].astype(np.float64) * 2.0 ** 24)
    n = len(u)
    if n < 3:
        return (0.0, 0.0, 0.0, 0.0)
    r0, r1, r2_ = _philox(attempts, uid)

    def below(r, k):
        return (((r >> np.uint64(32)) * np.uint64(k)) >> np.uint64(32)).astype(np.int64)

    i0, i1, i2 = below(r0, n), below(r1, n - 1), below(r2_, n - 2)
    i1 = i1 + (i1 >= i0)
    lo, hi = np.minimum(i0, i1), np.maximum(i0, i1)
    i2 = i2 + (i2 >= lo)
    i2 = i2 + (i2 >= hi)
    x0, x1, x2, y0, y1, y2 = u[i0], u[i1], u[i2], v[i0], v[i1], v[i2]
    D = 2 * (x0 * (y1 - y2) + x1 * (y2 - y0) + x2 * (y0 - y1))
    ok = D != 0
    Df = np.where(ok, D, 1).astype(np.float64)
    z0, z1, z2 = x0 * x0 + y0 * y0, x1 * x1 + y1 * y1, x2 * x2 + y2 * y2
    cx = (z0 * (y1 - y2) + z1 * (y2 - y0) + z2 * (y0 - y1)) / Df
    cy = (z0 * (x2 - x1) + z1 * (x0 - x2) + z2 * (x1 - x0)) / Df
    rr = (x0 - cx) ** 2 + (y0 - cy) ** 2
    uf, vf = u.astype(np.float64), v.astype(np.float64)
    z = uf * uf + vf * vf
    M = np.stack([np.ones(n), uf, vf, uf * uf, uf * vf, vf * vf, uf * z, vf * z], axis=1)

    def band():
        du, dv = uf[None, :] - cx[:, None], vf[None, :] - cy[:, None]
        d2, r = du * du + dv * dv, np.sqrt(rr)
        low = np.where(r > p.t_ri, (r - p.t_ri) ** 2, -1.0)
        return ((low[:, None] <= d2) & (d2 <= ((r + p.t_ri) ** 2)[:, None])).astype(np.float64)

    for _ in range(p.refine_iters):
        m, su, sv, suu, suv, svv, suz, svz = (band() @ M).T
        sz = suu + svv
        i64 = [t.astype(np.int64) for t in (m, su, sv, suu, suv, svv, suz, svz, sz)]
        im, isu, isv, isuu, isuv, isvv, isuz, isvz, isz = i64
        cuu, cuv, cvv = im * isuu - isu * isu, im * isuv - isu * isv, im * isvv - isv * isv
        cuz, cvz = im * isuz - isu * isz, im * isvz - isv * isz
        cuu, cuv, cvv, cuz, cvz = (t.astype(np.float64) for t in (cuu, cuv, cvv, cuz, cvz))
        det = cuu * cvv - cuv * cuv
        ok = ok & (m >= 3) & (det != 0)
        det = np.where(ok, det, 1.0)
        m = np.where(ok, m, 1.0)
        cx = np.where(ok, (cuz * cvv - cvz * cuv) / det / 2.0, 0.0)
        cy = np.where(ok, (cvz * cuu - cuz * cuv) / det / 2.0, 0.0)
        rr = (cuu + cvv) / (m * m) + (su / m - cx) ** 2 + (sv / m - cy) ** 2
    total = band() @ q
    ax, ay, r = W // 2 + cx, H // 2 + cy, np.sqrt(rr)
    off = (ax - (W - 1) / 2.0) ** 2 + (ay - (H - 1) / 2.0) ** 2
    ok = ok & (r >= p.r_min * W) & (r <= p.r_max * W) & (off <= (p.d_max * W) ** 2)
    if not ok.any():
        return (0.0, 0.0, 0.0, 0.0)
    b = int(np.argmax(np.where(ok, total, -1.0)))
    return (ax[b], ay[b], r[b], total[b] / (2.0 ** 24 * len(x)))


def _exact_circles(frames, case, uids):
    tables = _score_tables()
    out = []
    for f, uid in zip(frames, uids):
        a = f.cpu().numpy()
        out.append(_circle(_candidates(a, case["hs"], case["vs"], tables), a.shape[1], a.shape[0],
                           case["attempts"], uid))
    return np.array(out, dtype=np.float64)


# The two networks in float64 on plain tensors: the master weights, no
# rounding of weights or activations.

def _conv(x, w):
    """x [n, cin, lines, positions] (already padded), w [cout, cin, kl, kp]."""
    co, ci, kl, kp = w.shape
    n, _, ln, ps = x.shape
    ol, op = ln - kl + 1, ps - kp + 1
    xt = x.permute(0, 2, 3, 1)
    y = 0
    for a in range(kl):
        for b in range(kp):
            part = xt[:, a:a + ol, b:b + op].reshape(-1, ci)
            y = y + part @ w[:, :, a, b].t().contiguous()
    return y.reshape(n, ol, op, co).permute(0, 3, 1, 2)


def _take(flat, *shape):
    k = int(np.prod(shape))
    return flat[:k].reshape(shape), flat[k:]


def _net_1d(flat, win, rng_):
    """Logits [n, 112]."""
    n = win.shape[0]
    p = torch.arange(128, device=win.device)
    mask = ((p >= rng_[:, :1]) & (p < rng_[:, 1:])).to(torch.float64)[:, None, None, :]
    x = (win.to(torch.float64) - 128.0) / 64.0
    x = x.permute(0, 1, 3, 2).reshape(n, 24, 1, 128) * mask
    rest = flat
    for ci, co in ((24, 16), (16, 32), (32, 32), (32, 16)):
        w, rest = _take(rest, co, ci, 1, 5)
        b, rest = _take(rest, co)
        x = _conv(torch.nn.functional.pad(x, (2, 2)), w) + b[None, :, None, None]
        x = torch.relu(x) * mask
    w, rest = _take(rest, 16)
    b, rest = _take(rest, 1)
    z = (x * w[None, :, None, None]).sum(1)[:, 0] + b
    return z[:, 8:120]


def _net_2d(flat, win, geom, rng_):
    """Logits [n, 112]; every window of one orientation."""
    n = win.shape[0]
    dev = win.device
    mean, rest = _take(flat, 3)
    inv, rest = _take(rest, 3)
    g = geom.to(torch.int64)
    hz = bool(g[0, 0] != 0)
    line, start, W, H = (g[:, k] for k in (1, 2, 3, 4))
    p, j = torch.arange(128, device=dev), torch.arange(7, device=dev)
    across = line[:, None] - 3 + j[None, :]
    extent = H if hz else W
    lines = ((across >= 0) & (across < extent[:, None])).to(torch.float64)
    inside = ((p >= rng_[:, :1]) & (p < rng_[:, 1:])).to(torch.float64)
    mask = lines[:, :, None] * inside[:, None, :]
    colour = (win[:, :7].to(torch.float64) - mean) * inv
    along = (start[:, None] + p[None, :])[:, None, :].expand(n, 7, 128)
    acr = across[:, :, None].expand(n, 7, 128)
    xx, yy = (along, acr) if hz else (acr, along)
    cx = (2 * xx - (W - 1)[:, None, None]) / (2.0 * (W - 1)[:, None, None])
    cy = (2 * yy - (H - 1)[:, None, None]) / (2.0 * (H - 1)[:, None, None])
    x = torch.cat([colour.permute(0, 3, 1, 2), cx[:, None], cy[:, None]], 1) * mask[:, None]
    for k, (ci, co) in enumerate(((5, 8), (8, 16), (16, 32))):
        w, rest = _take(rest, co, ci, 3, 3)
        b, rest = _take(rest, co)
        w = w if hz else w.transpose(2, 3)
        x = _conv(torch.nn.functional.pad(x, (1, 1)), w) + b[None, :, None, None]
        x = torch.relu(x) * mask[:, None, k + 1:6 - k]
    w, rest = _take(rest, 32)
    b, rest = _take(rest, 1)
    z = (x[:, :, 0] * w[None, :, None]).sum(1) + b
    return z[:, 8:120]


def _exact_windows(case, seed):
    recs, desc = _window_batch(case, seed)
    b = train_scorer.Batch(recs, desc, 0.0, case["net"])
    two = case["net"] == "2d"
    flat = torch.from_numpy(_window_model(case).astype(np.float64)).to(b.win.device)
    train = case["kind"] == "train"
    flat.requires_grad_(train)
    n = b.win.shape[0]
    logits = torch.empty((n, 112), dtype=torch.float64, device=b.win.device)
    loss_sum = 0.0
    groups = [torch.arange(n, device=b.win.device)]
    if two:
        hz = b.geom[:, 0] != 0
        groups = [torch.nonzero(hz)[:, 0], torch.nonzero(~hz)[:, 0]]
    with torch.set_grad_enabled(train):
        for g in groups:
            for k in range(0, len(g), 1024):
                i = g[k:k + 1024]
                r = b.rng[i].to(torch.int64)
                z = (_net_2d(flat, b.win[i], b.geom[i], r) if two
                     else _net_1d(flat, b.win[i], r))
                if not train:
                    logits[i] = z
                    continue
                p = torch.arange(8, 120, device=z.device)
                here = ((p >= r[:, :1]) & (p < r[:, 1:])).to(torch.float64)
                t, wt = b.tgt[i].to(torch.float64), b.wt[i].to(torch.float64) * here
                soft = torch.clamp(z, min=0) - z * t + torch.log1p(torch.exp(-z.abs()))
                part = (wt * soft).sum() * b.scale
                part.backward()
                loss_sum += float(part.detach())
    if not train:
        return {"logits": logits}
    grad = flat.grad.clone()
    if two:
        grad[:6] = 0      # the normaliser is not trained
    return {"grad": grad, "loss": torch.tensor([loss_sum], dtype=torch.float64)}


def exact(case, seed):
    if case["kind"] in ("logits", "train"):
        return _exact_windows(case, seed)
    if case["scorer"] != 0:
        return None     # the best pixel of a bfloat16 network has no 64-bit value
    if case["kind"] == "estimate":
        return {"circle": _exact_circles(_frames(case, seed), case, range(case["n"])),
                "counts": None}
    frames = _streams(case, seed)
    c = _exact_circles(frames, case, [sid << 32 for sid in range(len(frames))])
    threshold = api.default_params().t_cs
    valid = (c[:, 3] >= threshold)[:, None]
    # the first frame of a stream is its filtered circle when it is valid
    return {"circle": c, "counts": None, "filtered": np.where(valid, c, 0.0)}
