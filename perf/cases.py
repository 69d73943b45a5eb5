"""Cases by which the filter's speed is measured on one GPU.

A case is a dict of plain values.  `prepare` makes what a program that uses the
filter has in hand before a call, `run` makes one pass through the package's
entry points, `work` says what the pass cannot do without, and `exact` says
what it returns, computed in plain torch without the package.

Kinds of case:
  frame      one frame of an animation through FrameFilter.  The state holds
             two frames of an orbiting camera; the first has been filtered
             already and the passes alternate between them, so every pass
             blends against the other frame's table as a renderer does.
  keys       insert and lookup of a stream of incoherent keys at a given
             table load (clear, binned insert, lookup).
  mlp_train  one training step of the learned fallback.
  mlp_infer  the learned fallback's selection of vertices and its inference.
  views      one frame of several views through MultiViewFilter.
"""
import math

import torch

import paper_1902_05942_amd as pf
import synth
from synth.mlp_init import init_params
from synth.scene import camera_position, generate_view, make_scene
from synth.workloads import frame_seed

ALPHA = 0.2  # weight of the previous frame's value, as the named workloads have it
SCALE = 0.01
MAX_PROBE, FRAC_BITS = 64, 24
SPARSE_BELOW, TRAIN_FROM, LEARNING_RATE = 4, 16, 1e-3
STEP_SEED = 0x9E3779B97F4A7C15


def log2_slots(pixels):
    """The named workloads' table size: the power of two at or above twice the pixels."""
    return min(25, max(14, (2 * pixels - 1).bit_length()))


def frame_case(width, height, verts, **options):
    case = {"kind": "frame", "width": width, "height": height, "verts": verts, "log2_slots": log2_slots(width * height),
            "scene": "boxes", "insert": "fused", "agg": 0, "float_sums": False, "max_samples": 0, "low_density": 0,
            "history": 0, "resolve": False}
    case.update(options)
    return case


def listed():
    return [
        # the smallest workload of the repository (its smoke test): launches and host time count
        dict(frame_case(64, 64, 1), name="frame_64x64"),
        # a small ragged image, as a preview or a tile of a larger one has it
        dict(frame_case(401, 229, 3), name="frame_401x229_x3"),
        # the benchmark's workload
        dict(frame_case(1920, 1080, 3, log2_slots=22), name="frame_1080p_x3"),
        # the largest single view: boxes and spheres, heavier noise
        dict(frame_case(3840, 2160, 4, scene="spheres"), name="frame_4k_x4"),
        # temporal integration, neighbourhood search for sparse cells, and the image formed from the result
        dict(frame_case(1280, 720, 3, max_samples=64, low_density=4, resolve=True), name="frame_720p_x3_sparse_resolve"),
        # the paper's own accumulation: binary32 sums, atomics combined over 64 lanes
        dict(frame_case(1280, 720, 3, insert="atomic", agg=64, float_sums=True), name="frame_720p_x3_float"),
        # separate key construction and binned insert, voxels remembered beyond the previous frame
        dict(frame_case(1280, 720, 3, insert="binned", history=21), name="frame_720p_x3_history"),
        # incoherent keys at a half-full table (the load sweep of the 4K workload, a smaller table)
        {"name": "keys_8m_load50", "kind": "keys", "n": 8 << 20, "log2_slots": 22, "load": 0.5},
        # one step of the learned fallback's online training at its default batch
        {"name": "mlp_train_16384", "kind": "mlp_train", "width": 1920, "height": 1080, "verts": 3, "batch": 16384},
        # the learned fallback's selection and inference for the benchmark's frame
        {"name": "mlp_infer_1080p_x3", "kind": "mlp_infer", "width": 1920, "height": 1080, "verts": 3},
        # a few small views in one persistent launch
        {"name": "views_4_persistent", "kind": "views", "mode": "persistent", "verts": 3,
         "sizes": "640x360,800x600,401x229,256x256"},
        # the eight uneven views of the multi-view workload on library streams
        {"name": "views_8_concurrent", "kind": "views", "mode": "concurrent", "verts": 3,
         "sizes": "640x360,1280x720,1920x1080,1920x1080,1920x1080,2560x1440,3840x2160,800x600"},
    ]


def draw(rng):
    def size(lo, hi):  # an image of lo .. hi pixels (over the logarithm), of any ordinary shape
        pixels = math.exp(rng.uniform(math.log(lo), math.log(hi)))
        width = max(16, int(math.sqrt(pixels * rng.uniform(0.8, 2.4))))
        return width, max(16, int(pixels / width))

    what = rng.choice(["fused", "fused", "fused", "sparse", "float", "history", "keys", "train", "infer", "persistent",
                       "concurrent"])
    if what == "fused":
        w, h = size(4096, 8 << 20)
        return frame_case(w, h, rng.randint(1, 4) if w * h > 6400 else rng.randint(1, 3),
                          scene=rng.choice(["boxes", "spheres"]), max_samples=rng.choice([0, 0, 32]))
    if what in ("sparse", "float", "history"):
        w, h = size(60000, 2 << 20)
        verts = rng.randint(1, 3)
        if what == "sparse":
            return frame_case(w, h, verts, max_samples=rng.choice([0, 64]), low_density=rng.randint(3, 6),
                              resolve=rng.random() < 0.5)
        if what == "float":
            return frame_case(w, h, verts, insert="atomic", agg=rng.choice([0, 64, 64, 256]),
                              float_sums=rng.random() < 0.5)
        return frame_case(w, h, verts, insert=rng.choice(["binned", "fused"]), history=rng.randint(18, 22))
    if what == "keys":
        m = rng.randint(18, 23)
        return {"kind": "keys", "n": int((1 << m) * rng.uniform(0.7, 2.0)), "log2_slots": m,
                "load": round(rng.uniform(0.1, 0.5), 3)}
    if what in ("train", "infer"):
        w, h = size(100000, 2 << 20)
        case = {"kind": "mlp_" + what, "width": w, "height": h, "verts": rng.randint(1, 3)}
        return dict(case, batch=64 * rng.randint(16, 512)) if what == "train" else case
    sizes = [size(16000, 1 << 19 if what == "persistent" else 2 << 20) for _ in range(rng.randint(2, 6))]
    return {"kind": "views", "mode": what, "verts": rng.randint(1, 3), "sizes": ",".join("%dx%d" % s for s in sizes)}


# ------------------------------------------------------------------ inputs
def frames_of(width, height, verts, scene, seed, numbers, device="cuda"):
    """Frames of the orbiting camera: vertex streams on the GPU and the filter's parameters."""
    spheres = scene == "spheres"
    sc = make_scene(seed, 64, 16, (0.2, 0.8)) if spheres else make_scene(seed, 8)
    out = []
    for k in numbers:
        f = generate_view(sc, width, height, verts, camera_position(k), seed, k, 1.5 if spheres else 1.0,
                          0.01 if spheres else 0.0, device=device)
        f = {x: f[x] for x in ("px", "py", "pz", "nx", "ny", "nz", "valid", "r", "g", "b", "tr", "tg", "tb", "cam")}
        f.update(seed=frame_seed(seed, k), s=SCALE)
        out.append(f)
    return out


def view_sizes(case):
    return [tuple(int(x) for x in s.split("x")) for s in case["sizes"].split(",")]


def prepare_frame(case, seed):
    frames = frames_of(case["width"], case["height"], case["verts"], case["scene"], seed, (0, 1))
    pixels = case["width"] * case["height"]
    n = pixels * case["verts"]
    flt = pf.FrameFilter(n, case["log2_slots"], MAX_PROBE, FRAC_BITS, temporal=True, alpha_old=ALPHA,
                         agg_width=case["agg"], binned=case["insert"] == "binned", fused=case["insert"] == "fused",
                         float_sums=case["float_sums"], max_samples=case["max_samples"] or None,
                         low_density=(case["low_density"], pf.LD_NEIGHBOURS) if case["low_density"] else None,
                         history=(case["history"], 8) if case["history"] else None)
    out = tuple(torch.empty(n, device="cuda") for _ in range(3))
    image = tuple(torch.empty(pixels, device="cuda") for _ in range(3)) if case["resolve"] else None
    state = {"case": case, "frames": frames, "filter": flt, "out": out, "image": image, "next": 0}
    run_frame(state)
    return state


def run_frame(state):
    case, flt, out = state["case"], state["filter"], state["out"]
    f = state["frames"][state["next"]]
    state["next"] ^= 1
    flt.filter(f["px"], f["py"], f["pz"], f["nx"], f["ny"], f["nz"], f["valid"], f["r"], f["g"], f["b"], f["cam"],
               f["s"], f["seed"], out=out, with_count=True)
    got = {"rgb": list(out), "count": flt.count, "flags": flt.vflags}
    if case["resolve"]:
        pf.resolve_pixels(*out, (f["tr"], f["tg"], f["tb"]), f["valid"], case["width"] * case["height"], case["verts"],
                          state["image"])
        got["image"] = list(state["image"])
    return got


def prepare_keys(case, seed):
    n = case["n"]
    s = synth.synthetic_keys(n, int(case["load"] * (1 << case["log2_slots"])), seed, device="cuda")
    table = pf.Table(case["log2_slots"], MAX_PROBE, FRAC_BITS, with_blend=False)
    pf.table_init(table)
    return {"case": case, "in": s, "table": table, "flags": torch.zeros(n, dtype=torch.uint8, device="cuda"),
            "slot": torch.empty(n, dtype=torch.int32, device="cuda"),
            "count": torch.empty(n, dtype=torch.int32, device="cuda"),
            "out": [torch.empty(n, device="cuda") for _ in range(3)],
            "ws": torch.empty(pf.insert_workspace_bytes(n, case["log2_slots"]), dtype=torch.uint8, device="cuda")}


def run_keys(st):
    s, out = st["in"], st["out"]
    pf.clear(st["table"])
    pf.insert_accumulate_binned(st["table"], s["key"], s["r"], s["g"], s["b"], st["flags"], st["slot"], st["ws"])
    pf.query_average(st["table"], s["key"], st["slot"], s["r"], s["g"], s["b"], st["flags"], False, *out, st["count"])
    return {"rgb": list(out), "count": st["count"], "flags": st["flags"]}


def prepare_mlp(case, seed):
    f = frames_of(case["width"], case["height"], case["verts"], "boxes", seed, (0,))[0]
    pixels = case["width"] * case["height"]
    n, m = pixels * case["verts"], log2_slots(pixels)
    table = pf.Table(m, MAX_PROBE, FRAC_BITS, with_blend=False)
    pf.table_init(table)
    key = torch.empty(n, dtype=torch.int64, device="cuda")
    slot, count = (torch.empty(n, dtype=torch.int32, device="cuda") for _ in range(2))
    flags = torch.empty(n, dtype=torch.uint8, device="cuda")
    out = [torch.empty(n, device="cuda") for _ in range(3)]
    ws = torch.empty(pf.insert_workspace_bytes(n, m), dtype=torch.uint8, device="cuda")
    pf.build_keys_insert_binned(table, f["px"], f["py"], f["pz"], f["nx"], f["ny"], f["nz"], f["valid"], f["cam"],
                                f["s"], f["seed"], 0, f["r"], f["g"], f["b"], key, flags, slot, ws)
    pf.query_average(table, key, slot, f["r"], f["g"], f["b"], flags, False, *out, count)
    fallback = pf.MlpFallback(n, init_params(seed), batch=case.get("batch", 16384), steps=1, lr=LEARNING_RATE,
                              sparse_below=SPARSE_BELOW, train_from=TRAIN_FROM)
    geo = pf.geometry(key, f["px"], f["py"], f["pz"], f["nx"], f["ny"], f["nz"], f["cam"])
    state = {"case": case, "frame": f, "table": table, "geo": geo, "slot": slot, "count": count, "flags": flags,
             "out": out, "fallback": fallback, "step": 0}
    select(state)
    return state


def select(st):
    fb = st["fallback"]
    pf.mlp_select(st["flags"], st["count"], fb.sparse_below, fb.train_from, fb.train_idx, fb.sparse_idx, fb.counts,
                  fb.ws)


def run_train(st):
    fb = st["fallback"]
    st["step"] += 1
    pf.mlp_train_step(fb.net, st["table"], st["geo"], st["slot"], fb.train_idx, fb.counts, fb.batch,
                      (st["frame"]["seed"] ^ (st["step"] * STEP_SEED)) & (2 ** 64 - 1), fb.lr)
    m, v = fb.net.moments()
    return {"weights": fb.net.weights(), "m": m, "v": v, "loss": fb.net.loss()}


def run_infer(st):
    fb = st["fallback"]
    select(st)
    pf.mlp_infer(fb.net, st["geo"], fb.sparse_idx, fb.counts, *st["out"])
    return {"rgb": list(st["out"]), "selected": fb.counts}


def prepare_views(case, seed):
    sizes = view_sizes(case)
    flt = pf.MultiViewFilter([(w * h * case["verts"], log2_slots(w * h)) for w, h in sizes], MAX_PROBE, FRAC_BITS,
                             alpha_old=ALPHA, keys=False, mode=case["mode"])
    frames = [frames_of(w, h, case["verts"], "boxes", seed + v, (0, 1)) for v, (w, h) in enumerate(sizes)]
    state = {"case": case, "filter": flt, "frames": frames, "next": 0}
    run_views(state)
    return state


def run_views(st):
    flt, k = st["filter"], st["next"]
    st["next"] ^= 1
    frames = [f[k] for f in st["frames"]]
    if st["case"]["mode"] == "persistent":
        out = flt.filter(frames, block=1024, agg_width=4096, with_count=True)  # the tuner's choice
    else:
        out = flt.filter(frames, with_count=True, nstreams=2)
    return [{"rgb": list(o), "count": b["count"], "flags": b["vflags"]} for o, b in zip(out, flt.bufs)]


def prepare(case, seed):
    make = {"frame": prepare_frame, "keys": prepare_keys, "mlp_train": prepare_mlp, "mlp_infer": prepare_mlp,
            "views": prepare_views}
    return make[case["kind"]](case, seed)


def run(state):
    go = {"frame": run_frame, "keys": run_keys, "mlp_train": run_train, "mlp_infer": run_infer, "views": run_views}
    return go[state["case"]["kind"]](state)


# -------------------------------------------------------------------- work
def frame_work(pixels, verts, cells_kept=1.0):
    """A frame reads one byte a slot, position, normal and contribution of each vertex that exists, writes value,
    count and flag of every slot (an empty slot's value is the input's), and reads and writes one record of 64 bytes
    a cell; about 0.95 of the primary vertices and a quarter of the others exist, a cell holds about 8 of them."""
    slots = pixels * verts
    live = pixels * (0.95 + 0.25 * (verts - 1))
    cells = live / 8 * cells_kept
    return {"bytes": slots * (1 + 12 + 4 + 1) + live * 36 + (slots - live) * 12 + cells * 128, "flops": 100.0 * live}


def work(case):
    kind = case["kind"]
    if kind == "frame":
        pixels = case["width"] * case["height"]
        w = frame_work(pixels, case["verts"])
        if case["resolve"]:
            w["bytes"] += pixels * (case["verts"] * 25 + 12)
        if case["history"]:
            w["bytes"] += (36 << case["history"])
        return w
    if kind == "keys":
        n, cells = case["n"], case["load"] * (1 << case["log2_slots"])
        return {"bytes": n * (8 + 12 + 1 + 4 + 12 + 4) + cells * 64, "flops": 30.0 * n}
    if kind == "mlp_train":
        # a sample's key, geometry and target; the weights and moments in and out
        return {"bytes": case["batch"] * (4 + 8 + 24 + 4 + 32) + 10384 * (4 * 6 + 2), "flops": 51200.0 * case["batch"]}
    if kind == "mlp_infer":
        n = case["width"] * case["height"] * case["verts"]
        sparse = 0.05 * n
        return {"bytes": n * 5 + sparse * (4 + 8 + 24 + 12) + 0.3 * n * 4, "flops": 2.0 * 10240 * sparse}
    total = {"bytes": 0.0, "flops": 0.0}
    for w, h in view_sizes(case):
        for k, v in frame_work(w * h, case["verts"]).items():
            total[k] += v
    return total


# ------------------------------------------------------------------- exact
def signed(x):
    x &= 2 ** 64 - 1
    return x - 2 ** 64 if x >= 2 ** 63 else x


def shr(x, k):
    return (x >> k) & ((1 << (64 - k)) - 1)


PCG = 6364136223846793005


def pcg_outputs(seed, streams, count):
    """First outputs of PCG32 (XSH-RR) for each stream."""
    inc = 2 * streams + 1
    state = (inc + signed(seed)) * PCG + inc
    for _ in range(count):
        x = shr(shr(state, 18) ^ state, 27) & 0xFFFFFFFF
        rot = shr(state, 59)
        yield ((x >> rot) | (x << ((32 - rot) & 31))) & 0xFFFFFFFF
        state = state * PCG + inc


def power_of_two(level):
    return ((level + 127) << 23).to(torch.int32).view(torch.float32)


def level_of(cam, x):
    d = [c - v for c, v in zip(cam, x)]
    d2 = (d[0] * d[0] + d[1] * d[1]) + d[2] * d[2]
    e = (d2.view(torch.int32) >> 23) & 0xFF
    level = torch.clamp((e - 127) >> 1, -16, 15)
    return torch.where(e == 0, -16, torch.where(e == 255, 15, level))


def keys_of(f):
    """Key of every vertex (-1: unfiltered): the binary32 steps of key construction, whose results are whole numbers."""
    x, n = [f[c] for c in ("px", "py", "pz")], [f[c] for c in ("nx", "ny", "nz")]
    stream = torch.arange(x[0].numel(), device=x[0].device)
    r = [(u >> 8).to(torch.float32) * 2.0 ** -24 - 0.5 for u in pcg_outputs(f["seed"], stream, 3)]
    t = (r[0] * n[0] + r[1] * n[1]) + r[2] * n[2]
    s = torch.tensor(f["s"], dtype=torch.float32, device=x[0].device)
    h = s * power_of_two(level_of(f["cam"], x))
    x = [xc + (rc - t * nc) * h for xc, rc, nc in zip(x, r, n)]
    level = level_of(f["cam"], x)
    h = s * power_of_two(level)
    q = [torch.floor((xc.double() / h.double()).float()) for xc in x]
    ok = f["valid"] != 0
    for v in q:
        ok &= v.abs() < 65536
    key = (level.to(torch.int64) + 16) << 51
    for c in range(3):
        key |= (torch.where(ok, q[c], 0.0).to(torch.int64) + 65536) << (17 * c)
        key |= torch.where(n[c] > 0, 1, torch.where(n[c] < 0, 2, 0)) << (56 + 2 * c)
    return torch.where(ok, key, -1)


class Cells:
    """The cells of a stream of keys: sorted keys, counts, sums in 64 bits, each vertex's cell."""

    def __init__(self, key, rgb):
        self.ok = key >= 0
        self.key, self.of = torch.unique(key[self.ok], return_inverse=True)
        self.count = torch.bincount(self.of, minlength=self.key.numel())
        self.sum = torch.zeros(self.key.numel(), 3, dtype=torch.float64, device=key.device)
        for c in range(3):
            self.sum[:, c].index_add_(0, self.of, rgb[c][self.ok].double())
        self.value = self.sum / self.count[:, None]
        self.kept = self.count.clone()  # the count stored with the value

    def find(self, key):
        at = torch.searchsorted(self.key, key).clamp(max=self.key.numel() - 1)
        return at, self.key[at] == key

    def blend(self, old, max_samples, seen=None):
        if max_samples:
            self.kept = self.kept.clamp(max=max_samples)
        if old is None:
            return
        at, hit = old.find(self.key)
        if seen is not None:
            hit &= seen[at]
        a = torch.full_like(self.value[:, 0], ALPHA)
        if max_samples:
            total = old.kept[at] + self.count
            a = old.kept[at].double() / total.double()
            self.kept = torch.where(hit, total.clamp(max=max_samples), self.kept)
        mixed = a[:, None] * old.value[at] + (1 - a)[:, None] * self.value
        self.value = torch.where(hit[:, None], mixed, self.value)

    def pool_sparse(self, below):
        """Cells with fewer vertices take the average over the 27 cells around them."""
        few = torch.nonzero(self.count < below)[:, 0]
        key = self.key[few]
        base = key & ~((1 << 51) - 1)
        x = [((key >> (17 * a)) & 0x1FFFF) - 65536 for a in range(3)]
        total, count = torch.zeros_like(self.sum[few]), torch.zeros_like(self.count[few])
        for c in range(27):
            y = [v + d for v, d in zip(x, (c % 3 - 1, c // 3 % 3 - 1, c // 9 - 1))]
            near = base | (y[0] + 65536) | ((y[1] + 65536) << 17) | ((y[2] + 65536) << 34)
            at, hit = self.find(near)
            for v in y:
                hit &= v.abs() < 65536
            total += torch.where(hit[:, None], self.sum[at], 0.0)
            count += torch.where(hit, self.count[at], 0)
        self.value[few] = total / count[:, None]

    def in_history(self, log2):
        """Which cells a direct-mapped history keeps of one frame: of a slot's cells the smallest word."""
        k = self.key ^ shr(self.key, 33)
        k = k * signed(0xFF51AFD7ED558CCD)
        k = k ^ shr(k, 33)
        k = k * signed(0xC4CEB9FE1A85EC53)
        slot = (k ^ shr(k, 33)) & ((1 << log2) - 1)
        z = self.key + signed(0x9E3779B97F4A7C15)
        z = (z ^ shr(z, 30)) * signed(0xBF58476D1CE4E5B9)
        z = (z ^ shr(z, 27)) * signed(0x94D049BB133111EB)
        lg = torch.log2(self.kept.double() + 0.25).floor().to(torch.int64).clamp(max=15)
        word = ((15 - lg) << 56) | ((z ^ shr(z, 31)) & ((1 << 56) - 1))
        least = torch.full((1 << log2,), 2 ** 62, dtype=torch.int64, device=word.device)
        least.scatter_reduce_(0, slot, word, "amin")
        return least[slot] == word

    def lookup(self, rgb):
        out = [c.double().clone() for c in rgb]
        for c in range(3):
            out[c][self.ok] = self.value[self.of, c]
        count = torch.zeros(self.ok.numel(), dtype=torch.int32, device=self.ok.device)
        count[self.ok] = self.kept[self.of].to(torch.int32)
        return out, count


def exact_frame(frames, max_samples=0, low_density=0, history=0):
    old = seen = None
    for f in frames:
        rgb = (f["r"], f["g"], f["b"])
        key = keys_of(f)
        cells = Cells(key, rgb)
        cells.blend(old, max_samples, seen)
        if low_density:
            cells.pool_sparse(low_density)
        if history:
            seen = cells.in_history(history)
        old = cells
    out, count = cells.lookup(rgb)
    return {"rgb": out, "count": count, "flags": None if (key[f["valid"] != 0] < 0).any() else (f["valid"] == 0).to(torch.uint8)}


def features(f, key, v):
    """The network's 80 inputs of the vertices v."""
    k = key[v]
    lp = ((k >> 51) & 31) - 16
    cols = [None] * 80
    for j in range(12):
        for c in range(3):
            phase = (((k >> (17 * c)) & 0x1FFFF) - 65536 + 0.5).double() * torch.exp2((lp - 10 + j).double())
            phase = phase - 2 * torch.round(phase / 2)
            cols[6 * j + c], cols[6 * j + 3 + c] = torch.sin(math.pi * phase), torch.cos(math.pi * phase)
    d = [f[a][v].double() - cam for a, cam in zip(("px", "py", "pz"), f["cam"])]
    length = torch.sqrt(d[0] * d[0] + d[1] * d[1] + d[2] * d[2])
    cols[72:75] = [f[a][v].double() for a in ("nx", "ny", "nz")]
    cols[75:78] = [x / length for x in d]
    cols[78:80] = [torch.zeros_like(length)] * 2
    return torch.stack(cols, 1)


def network(seed, device):
    w = torch.from_numpy(init_params(seed)).to(device).double()
    at, out = 0, []
    for rows, columns in ((64, 80), (64, 1), (64, 64), (64, 1), (16, 64), (16, 1)):
        out.append(w[at:at + rows * columns].view(rows, columns).clone().requires_grad_())
        at += rows * columns
    return w, out


def predict(p, x):
    a = torch.relu(x @ p[0].t() + p[1].t())
    a = torch.relu(a @ p[2].t() + p[3].t())
    return (a @ p[4].t() + p[5].t())[:, :3]


def exact_mlp(case, seed):
    f = frames_of(case["width"], case["height"], case["verts"], "boxes", seed, (0,))[0]
    key = keys_of(f)
    cells = Cells(key, (f["r"], f["g"], f["b"]))
    out, count = cells.lookup((f["r"], f["g"], f["b"]))
    train = torch.nonzero(cells.ok & (count >= TRAIN_FROM))[:, 0]
    sparse = torch.nonzero(cells.ok & (count < SPARSE_BELOW))[:, 0]
    w, p = network(seed, key.device)
    if case["kind"] == "mlp_infer":
        with torch.no_grad():
            y = torch.cat([predict(p, features(f, key, part)) for part in torch.split(sparse, 1 << 18)] or [w[:0].view(0, 3)])
        for c in range(3):
            out[c][sparse] = y[:, c].clamp(min=0)
        return {"rgb": out, "selected": torch.tensor([train.numel(), sparse.numel()], dtype=torch.int32)}
    u = next(pcg_outputs(f["seed"] ^ STEP_SEED, torch.arange(case["batch"], device=key.device), 1))
    v = train[(u * train.numel()) >> 32]
    target = torch.stack([c[v] for c in out], 1)
    loss = ((predict(p, features(f, key, v)) - target) ** 2).mean()
    loss.backward()
    g = torch.cat([x.grad.reshape(-1) for x in p])
    m, s = 0.1 * g, 0.001 * g * g
    w = w - LEARNING_RATE * (m / 0.1) / (torch.sqrt(s / 0.001) + 1e-8)
    return {"weights": w, "m": m, "v": s, "loss": loss.detach().reshape(1)}


def exact(case, seed):
    """What the first `run` of a new state returns, in 64 bits."""
    kind = case["kind"]
    if kind == "frame":
        frames = frames_of(case["width"], case["height"], case["verts"], case["scene"], seed, (0, 1))
        got = exact_frame(frames, case["max_samples"], case["low_density"], case["history"])
        if case["resolve"]:
            f, shape = frames[1], (case["verts"], case["width"] * case["height"])
            live = f["valid"].view(shape) != 0
            got["image"] = [torch.where(live, f[t].double().view(shape) * c.view(shape), 0.0).sum(0)
                            for t, c in zip(("tr", "tg", "tb"), got["rgb"])]
        return got
    if kind == "keys":
        s = synth.synthetic_keys(case["n"], int(case["load"] * (1 << case["log2_slots"])), seed, device="cuda")
        out, count = Cells(s["key"], (s["r"], s["g"], s["b"])).lookup((s["r"], s["g"], s["b"]))
        return {"rgb": out, "count": count, "flags": torch.zeros(case["n"], dtype=torch.uint8)}
    if kind in ("mlp_train", "mlp_infer"):
        return exact_mlp(case, seed)
    return [exact_frame(frames_of(w, h, case["verts"], "boxes", seed + v, (0, 1)))
            for v, (w, h) in enumerate(view_sizes(case))]
