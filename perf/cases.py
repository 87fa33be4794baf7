"""What is timed: the calls that a program makes of this library at every camera step.

Each case is one pass through the public entry points, on inputs made on the GPU from a seed.
Frames are smooth coloured textures with hard-edged rectangles, the current frame being the
previous one moved by up to 20 pixels, with another brightness and sensor noise.  Hidden states
and caches are N(0, 1), weights N(0, 0.02), and the recomputed tokens a random ascending set,
another number of them for each item, as a selection leaves them.

Kinds of cases
  select   Algorithm 1 on a batch of frame pairs (fc_select), with the displacement from the token
           grid or from the full-resolution luma (align "pixel").
  carry    two consecutive camera steps of an episode with the spectra carried (fc_select_carry).
  phase    fc_phase_correlate alone, with its peak and its response surface.
  layer    one partial-recompute decoder layer (fc_layer_forward), on copied or slot-mapped rows.
  trail    the text after the frames through a decoder layer (fc_layer_forward_trail).
  remap    the cache remap of several decoder layers at once (fc_cache_update_layers).
  vit      one vision block over the recomputed patches (fc_vit_block_forward).
  vitmap   the encoder cache's remap from the previous frame's cache (fc_vit_cache_update).
  merger   the patch merger for the recomputed tokens (fc_vit_merger_forward).
  step     a whole camera step of a short model: selection, two vision blocks with their remaps,
           the merger, the decoder remap and two decoder layers.
"""
import math

import torch

import paper_2604_24391_amd as fc

P = 14
DEV = "cuda"

# Decoder blocks (d_model, query heads, kv heads, head dim, SwiGLU size): the Qwen2.5-VL-7B language
# block, the toy block, and small ones of the other head groupings the library is built for.
LAYERS = {"qwen": (3584, 28, 4, 128, 18944), "toy": (256, 4, 4, 64, 1024),
          "gqa7": (512, 7, 1, 128, 1024), "mha128": (512, 4, 4, 128, 1024),
          "gqa2": (512, 8, 4, 64, 1024), "gqa4": (512, 8, 2, 128, 1024)}
# Vision blocks (d_model, heads, head dim, MLP size): the Qwen2.5-VL block (its 3420 padded to a
# multiple of 64 with zeros) and a small one.
VITS = {"qwen": (1280, 16, 80, 3456), "small": (320, 4, 80, 448)}
MERGERS = {"qwen": (1280, 2, 3584), "small": (320, 2, 256)}
MROPE = (16, 24, 24)      # rotary pairs turned by the temporal, row and column position


def listed():
    return [
        # one small pair at a fixed budget, the smallest call: launches and latency
        dict(name="select_1x224", kind="select", items=1, h=224, w=224, merge=1, align="grid",
             adaptive=False),
        # a robot's episode: one 448 x 448 camera, 2 x 2 merge, spectra carried from step to step
        dict(name="carry_1x448", kind="carry", items=1, h=448, w=448, merge=2),
        # many robots at once: 64 independent pairs in one call
        dict(name="select_64x448", kind="select", items=64, h=448, w=448, merge=1, align="grid",
             adaptive=True),
        # the same with the displacement taken at pixel resolution
        dict(name="select_pixel_64x448", kind="select", items=64, h=448, w=448, merge=1,
             align="pixel", adaptive=True),
        # the toy block over 32 + 256 positions: a layer that is all launches
        dict(name="layer_toy", kind="layer", shape="toy", items=1, tokens=256, grid_w=16, window=1,
             text=32, mrope=False, slots=False, reuse=50),
        # a robot's decoder layer: 256 tokens a frame, 8 frames and 128 text tokens
        dict(name="layer_1x256", kind="layer", shape="qwen", items=1, tokens=256, grid_w=16, window=8,
             text=128, mrope=True, slots=False, reuse=37),
        # 16 episodes of large frames: the projections are compute bound
        dict(name="layer_16x1024", kind="layer", shape="qwen", items=16, tokens=1024, grid_w=32,
             window=4, text=128, mrope=True, slots=False, reuse=36),
        # the step's cache remap for every layer of the language model
        dict(name="remap_28_layers", kind="remap", shape="qwen", layers=28, items=1, tokens=256,
             grid_w=16, window=8, text=128, reuse=37),
        # a windowed vision block on a 448 x 448 frame at the mean reuse
        dict(name="vit_window_1x448", kind="vit", shape="qwen", items=1, grid_h=16, grid_w=16, merge=2,
             window=4, reuse=37),
        # a full-attention vision block with every token recomputed (a flushed step)
        dict(name="vit_full_1x448", kind="vit", shape="qwen", items=1, grid_h=16, grid_w=16, merge=2,
             window=0, reuse=0),
        # the merger behind it
        dict(name="merger_1x256", kind="merger", shape="qwen", items=1, tokens=256, reuse=37),
        # a whole step, frame in, hidden states out
        dict(name="step_1x448", kind="step", h=448, w=448, window=8, text=128),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["select", "select", "carry", "phase", "layer", "layer", "layer", "trail",
                       "remap", "vit", "vit", "vitmap", "merger", "step"])
    if kind in ("select", "carry"):
        align = "grid" if kind == "carry" else rng.choice(["grid", "grid", "pixel"])
        merge = rng.choice([1, 2])
        if align == "pixel":
            h, w = rng.choice([224, 448]), rng.choice([224, 448])
        else:
            most = 32 if merge == 1 else 16
            h, w = (P * merge * rng.randint(4, most) for _ in range(2))
        items = _log_int(rng, 1, 64) if kind == "select" else _log_int(rng, 1, 16)
        c = dict(kind=kind, items=items, h=h, w=w, merge=merge)
        if kind == "select":
            c.update(align=align, adaptive=rng.random() < 0.8)
        return c
    if kind == "phase":
        return dict(kind=kind, items=_log_int(rng, 1, 32), h=rng.choice([112, 224, 448, 896]),
                    w=rng.choice([112, 224, 448]))
    if kind in ("layer", "trail", "remap"):
        shape = rng.choice(["qwen", "qwen", "toy", "gqa7", "mha128", "gqa2", "gqa4"])
        gw = rng.randint(8, 32)
        gh = rng.randint(8, 32)
        window = rng.randint(2 if kind == "remap" else 1, 8 if gh * gw <= 512 else 4)
        c = dict(kind=kind, shape=shape, items=_log_int(rng, 1, 12), tokens=gh * gw, grid_w=gw,
                 window=window, text=rng.randint(16, 192))
        if kind == "remap":
            c.update(layers=rng.randint(1, 8) if c["items"] > 2 else rng.randint(1, 28),
                     reuse=rng.randint(8, 50))
        else:
            hd = LAYERS[shape][3]
            c.update(mrope=hd == 128 and rng.random() < 0.6)
            if kind == "trail":
                c.update(trail=rng.randint(3, 160))
            else:
                c.update(slots=rng.random() < 0.25, reuse=rng.choice([0, 25, 37, 50, 75, 90]))
        return c
    if kind in ("vit", "vitmap"):
        shape = rng.choice(["qwen", "qwen", "small"])
        c = dict(kind=kind, shape=shape, items=_log_int(rng, 1, 6), grid_h=rng.randint(4, 20),
                 grid_w=rng.randint(4, 20), merge=2, window=rng.choice([4, 4, 0]),
                 reuse=rng.choice([0, 25, 37, 50, 75, 90]))
        return c
    if kind == "merger":
        return dict(kind=kind, shape=rng.choice(["qwen", "qwen", "small"]), items=_log_int(rng, 1, 8),
                    tokens=rng.randint(16, 400), reuse=rng.choice([0, 25, 37, 50, 75, 90]))
    return dict(kind="step", h=28 * rng.randint(8, 18), w=28 * rng.randint(8, 18),
                window=rng.randint(2, 8), text=rng.randint(16, 160))


# ------------------------------------------------------------------------------------- inputs
def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed))
    return g


def _bf16(g, *shape, std=1.0):
    return torch.randn(*shape, device=DEV, generator=g, dtype=torch.bfloat16).mul_(std)


def _frames(g, n, h, w):
    """n frame pairs [n, 3, h, w] float32 in [0, 1]: a texture and its moved crop."""
    m = 32
    hh, ww = h + 2 * m, w + 2 * m
    tex = torch.zeros(n, 3, hh, ww, device=DEV)
    for cells, amp in ((6, 1.0), (18, 0.5), (48, 0.2)):
        grid = torch.rand(n, 3, cells, cells, device=DEV, generator=g)
        tex += amp * torch.nn.functional.interpolate(grid, size=(hh, ww), mode="bilinear",
                                                     align_corners=False)
    tex /= 1.7
    ys = torch.arange(hh, device=DEV).view(1, 1, hh, 1)
    xs = torch.arange(ww, device=DEV).view(1, 1, 1, ww)
    for _ in range(8):
        r = torch.rand(n, 7, 1, 1, 1, device=DEV, generator=g)
        y0, x0 = r[:, 0] * hh, r[:, 1] * ww
        inside = (ys >= y0) & (ys < y0 + P + 5 * P * r[:, 2]) & (xs >= x0) & (xs < x0 + P + 5 * P * r[:, 3])
        tex = torch.where(inside, r[:, 4:7, 0], tex)
    move = torch.randint(-20, 21, (n, 2), device=DEV, generator=g)
    gain = 0.9 + 0.2 * torch.rand(n, 1, 1, 1, device=DEV, generator=g)
    prev = tex[:, :, m:m + h, m:m + w].contiguous()
    iy = (m + torch.arange(h, device=DEV)).view(1, h) + move[:, 0:1]
    ix = (m + torch.arange(w, device=DEV)).view(1, w) + move[:, 1:2]
    cur = tex.gather(2, iy.view(n, 1, h, 1).expand(n, 3, h, ww))
    cur = cur.gather(3, ix.view(n, 1, 1, w).expand(n, 3, h, w))
    cur = cur * gain + 0.02 * torch.randn(n, 3, h, w, device=DEV, generator=g)
    return prev, cur.clamp_(0, 1)


def _reused(item, tokens, percent):
    """Tokens that item reuses: about percent of them, another number for each item."""
    p = percent + ((item * 7 + 3) % 11 - 5 if 0 < percent < 90 else 0)
    return tokens * p // 100


def _ids(g, items, tokens, percent):
    """recompute_idx [items, tokens], n_recompute [items] and reuse_mask [items, tokens]."""
    idx = torch.full((items, tokens), -1, dtype=torch.int32, device=DEV)
    mask = torch.zeros(items, tokens, dtype=torch.uint8, device=DEV)
    counts = []
    for b in range(items):
        k = _reused(b, tokens, percent)
        perm = torch.randperm(tokens, device=DEV, generator=g)
        mask[b, perm[:k]] = 1
        counts.append(tokens - k)
        idx[b, :tokens - k] = perm[k:].sort().values.int()
    return idx, torch.tensor(counts, dtype=torch.int32, device=DEV), mask


def _shifts(g, items, mask, gh, gw):
    """A displacement of up to two tokens for each item; a token without a source is not reused."""
    shift = torch.randint(-2, 3, (items, 2), device=DEV, generator=g, dtype=torch.int32)
    i = torch.arange(gh, device=DEV).view(1, gh, 1) + shift[:, 0].view(-1, 1, 1)
    j = torch.arange(gw, device=DEV).view(1, 1, gw) + shift[:, 1].view(-1, 1, 1)
    ok = (i >= 0) & (i < gh) & (j >= 0) & (j < gw)
    return shift, (mask * ok.reshape(items, gh * gw)).contiguous()


def _layer_weights(g, shape):
    d, nh, nkv, hd, f = LAYERS[shape]
    q = (nh + 2 * nkv) * hd
    return dict(w_qkv=_bf16(g, q, d, std=0.02), b_qkv=_bf16(g, q, std=0.02),
                w_o=_bf16(g, d, nh * hd, std=0.02), w_gate=_bf16(g, f, d, std=0.02),
                w_up=_bf16(g, f, d, std=0.02), w_down=_bf16(g, d, f, std=0.02),
                g_attn=_bf16(g, d, std=0.1).add_(1), g_mlp=_bf16(g, d, std=0.1).add_(1))


def _vit_weights(g, shape):
    d, _, _, f = VITS[shape]
    w = dict(w_qkv=_bf16(g, 3 * d, d, std=0.02), b_qkv=_bf16(g, 3 * d, std=0.02),
             w_o=_bf16(g, d, d, std=0.02), b_o=_bf16(g, d, std=0.02),
             w_gate_up=_bf16(g, 2 * f, d, std=0.02), b_gate_up=_bf16(g, 2 * f, std=0.02),
             w_down=_bf16(g, d, f, std=0.02), b_down=_bf16(g, d, std=0.02),
             g1=_bf16(g, d, std=0.1).add_(1), g2=_bf16(g, d, std=0.1).add_(1))
    if shape == "qwen":      # the rows past 3420 are padding
        for t in (w["w_gate_up"], w["b_gate_up"]):
            t[3420:f] = 0
            t[f + 3420:] = 0
        w["w_down"][:, 3420:] = 0
    return w


def _merger_weights(g, shape):
    d, m, o = MERGERS[shape]
    h = m * m * d
    return dict(g=_bf16(g, d, std=0.1).add_(1), w1=_bf16(g, h, h, std=0.02), b1=_bf16(g, h, std=0.02),
                w2=_bf16(g, o, h, std=0.02), b2=_bf16(g, o, std=0.02))


def _layer_desc(shape, w):
    d, nh, nkv, hd, f = LAYERS[shape]
    return fc.LayerDesc(d, nh, nkv, hd, f, w)


def _layer_caps(c, seq):
    d, nh, nkv, hd, f = LAYERS[c["shape"]]
    return fc.Caps(max_batch=c["items"], max_height=28, max_width=28,
                   max_tokens=max(c["tokens"], c.get("trail", 0)), max_seq=seq, max_d_model=d,
                   max_ffn=f, max_qkv=(nh + 2 * nkv) * hd)


def _layer_inputs(c, g):
    """Weights, cache and activations of a layer or trail case, by name."""
    d, nh, nkv, hd, f = LAYERS[c["shape"]]
    B, N, U = c["items"], c["tokens"], c.get("trail", 0)
    S = c["text"] + c["window"] * N + U
    t = dict(w=_layer_weights(g, c["shape"]), S=S, k=_bf16(g, B, S, nkv, hd), v=_bf16(g, B, S, nkv, hd))
    rows = U or N
    t["x"], t["y"] = _bf16(g, B, rows, d), _bf16(g, B, rows, d)
    if not U:
        t["idx"], t["nrec"], _ = _ids(g, B, N, c["reuse"])
    return t


def _vit_inputs(c, g):
    d, H, hd, f = VITS[c["shape"]]
    B, N = c["items"], c["grid_h"] * c["grid_w"]
    Np = N * c["merge"] ** 2
    t = dict(k=_bf16(g, B, Np, H, hd), v=_bf16(g, B, Np, H, hd), y=_bf16(g, B, Np, d))
    t["idx"], t["nrec"], mask = _ids(g, B, N, c["reuse"])
    if c["kind"] == "vit":
        t.update(w=_vit_weights(g, c["shape"]), x=_bf16(g, B, Np, d))
    else:
        t.update(k_prev=_bf16(g, B, Np, H, hd), v_prev=_bf16(g, B, Np, H, hd), y_prev=_bf16(g, B, Np, d))
        t["shift"], t["mask"] = _shifts(g, B, mask, c["grid_h"], c["grid_w"])
    return t


def _step_inputs(c, g):
    """Frames, weights and caches of a step case."""
    gh, gw = c["h"] // 28, c["w"] // 28
    N = gh * gw
    d, nh, nkv, hd, f = LAYERS["qwen"]
    vd, vH, vhd, vf = VITS["qwen"]
    S = c["text"] + c["window"] * N
    prev, cur = _frames(g, 1, c["h"], c["w"])
    t = dict(prev=prev, cur=cur, gh=gh, gw=gw, N=N, S=S, emb=_bf16(g, 1, 4 * N, vd), vit=[], lay=[])
    for win in (4, 0):
        t["vit"].append(dict(w=_vit_weights(g, "qwen"), win=win, kp=_bf16(g, 1, 4 * N, vH, vhd),
                             vp=_bf16(g, 1, 4 * N, vH, vhd), k=_bf16(g, 1, 4 * N, vH, vhd),
                             v=_bf16(g, 1, 4 * N, vH, vhd), y=_bf16(g, 1, 4 * N, vd)))
    t["mw"] = _merger_weights(g, "qwen")
    t["x"] = _bf16(g, 1, N, d)
    for _ in range(2):
        t["lay"].append(dict(w=_layer_weights(g, "qwen"), k=_bf16(g, 1, S, nkv, hd),
                             v=_bf16(g, 1, S, nkv, hd), yp=_bf16(g, 1, N, d), y=_bf16(g, 1, N, d)))
    return t


# ------------------------------------------------------------------------------------ prepare
def prepare(case, seed):
    c, g = case, _gen(seed)
    kind = c["kind"]
    s = dict(case=c)
    if kind in ("select", "carry", "phase"):
        B, h, w = c["items"], c["h"], c["w"]
        s["prev"], s["cur"] = _frames(g, B, h, w)
        tp = P * c.get("merge", 1)
        N = min(1024, (h // tp) * (w // tp))
        s["ctx"] = fc.Context(fc.Caps(max_batch=B, max_height=h, max_width=w, max_tokens=N, max_seq=16,
                                      max_d_model=64, max_ffn=64, max_qkv=192))
        if kind == "phase":
            s["shift_px"] = torch.zeros(B, 2, dtype=torch.float64, device=DEV)
            s["peak"] = torch.zeros(B, 2, dtype=torch.int32, device=DEV)
            s["resp"] = torch.zeros(B, h, w, dtype=torch.float64, device=DEV)
            return s
        s["prm"] = fc.SelectParams(merge=c["merge"], adaptive=c.get("adaptive", True),
                                   align_pixel=c.get("align") == "pixel")
        s["out"] = [fc.SelectOut.alloc(B, N) for _ in range(1 if kind == "select" else 2)]
        if kind == "carry":
            # the frame before, its spectra already carried; the step after goes back to its place
            s["states"] = [fc.select_state_alloc(B, h, w) for _ in range(3)]
            fc.fc_select_carry(s["ctx"], s["prm"], None, s["prev"], s["states"][0], s["out"][0])
        return s
    if kind in ("layer", "trail"):
        t = _layer_inputs(c, g)
        d, nh, nkv, hd, f = LAYERS[c["shape"]]
        s.update(t, ctx=fc.Context(_layer_caps(c, t["S"])), desc=_layer_desc(c["shape"], t["w"]))
        slot_map = fc.slot_state_alloc(c["items"], t["S"]) if c.get("slots") else None
        s["kv"] = fc.KVCache(t["k"], t["v"], c["text"], c["tokens"], c["window"], head=c["window"] // 2,
                             grid_w=c["grid_w"], mrope=MROPE if c["mrope"] else (0, 0, 0),
                             trail_tokens=c.get("trail", 0), slot_map=slot_map)
        if slot_map is not None:
            fc.fc_slot_map_init(s["ctx"], s["desc"], s["kv"], c["items"])
        return s
    if kind == "remap":
        d, nh, nkv, hd, f = LAYERS[c["shape"]]
        B, N, W = c["items"], c["tokens"], c["window"]
        S = c["text"] + W * N
        s["ctx"] = fc.Context(_layer_caps(c, S))
        # only the sizes of the weights matter to a remap: one layer's serve for all
        s["desc"] = _layer_desc(c["shape"], _layer_weights(g, c["shape"]))
        s["kvs"] = [fc.KVCache(_bf16(g, B, S, nkv, hd), _bf16(g, B, S, nkv, hd), c["text"], N, W,
                               head=W // 2) for _ in range(c["layers"])]
        s["yp"] = [_bf16(g, B, N, d) for _ in range(c["layers"])]
        s["yc"] = [_bf16(g, B, N, d) for _ in range(c["layers"])]
        _, _, mask = _ids(g, B, N, c["reuse"])
        s["shift"], s["mask"] = _shifts(g, B, mask, N // c["grid_w"], c["grid_w"])
        return s
    if kind in ("vit", "vitmap"):
        d, H, hd, f = VITS[c["shape"]]
        t = _vit_inputs(c, g)
        N = c["grid_h"] * c["grid_w"]
        mm = c["merge"] ** 2
        s.update(t, ctx=fc.Context(fc.Caps(max_batch=c["items"], max_height=28, max_width=28, max_tokens=N,
                                           max_seq=64, max_d_model=mm * d, max_ffn=mm * f,
                                           max_qkv=mm * d)))
        w = t["w"] if kind == "vit" else _vit_weights(g, c["shape"])
        s["desc"] = fc.VitDesc(d, H, hd, f, w)
        s["cache"] = fc.VitCache(t["k"], t["v"], c["grid_h"], c["grid_w"], c["merge"], c["window"],
                                 k_prev=t.get("k_prev"), v_prev=t.get("v_prev"))
        return s
    if kind == "merger":
        d, m, o = MERGERS[c["shape"]]
        B, N = c["items"], c["tokens"]
        s.update(_merger_inputs(c, g))
        s["ctx"] = fc.Context(fc.Caps(max_batch=B, max_height=28, max_width=28, max_tokens=N, max_seq=64,
                                      max_d_model=m * m * d, max_ffn=2 * m * m * d, max_qkv=m * m * d))
        s["desc"] = fc.MergerDesc(d, m, o, s["w"])
        return s
    t = _step_inputs(c, g)
    N, S, gh, gw = t["N"], t["S"], t["gh"], t["gw"]
    d, nh, nkv, hd, f = LAYERS["qwen"]
    vd, vH, vhd, vf = VITS["qwen"]
    s.update(t)
    s["ctx"] = fc.Context(fc.Caps(max_batch=1, max_height=c["h"], max_width=c["w"], max_tokens=N, max_seq=S,
                                  max_d_model=max(d, 4 * vd), max_ffn=max(f, 4 * vf), max_qkv=4 * vd))
    s["prm"] = fc.SelectParams(merge=2)
    s["sel"] = fc.SelectOut.alloc(1, N)
    s["states"] = [fc.select_state_alloc(1, c["h"], c["w"]) for _ in range(2)]
    fc.fc_select_carry(s["ctx"], s["prm"], None, t["prev"], s["states"][0], s["sel"])
    for b in s["vit"]:
        b["desc"] = fc.VitDesc(vd, vH, vhd, vf, b["w"])
        b["cache"] = fc.VitCache(b["k"], b["v"], gh, gw, 2, b["win"], k_prev=b["kp"], v_prev=b["vp"])
    s["merger"] = fc.MergerDesc(vd, 2, d, t["mw"])
    for b in s["lay"]:
        b["desc"] = _layer_desc("qwen", b["w"])
        b["kv"] = fc.KVCache(b["k"], b["v"], c["text"], N, c["window"], head=c["window"] // 2, grid_w=gw,
                             mrope=MROPE)
    return s


def _merger_inputs(c, g):
    d, m, o = MERGERS[c["shape"]]
    B, N = c["items"], c["tokens"]
    t = dict(w=_merger_weights(g, c["shape"]), y=_bf16(g, B, N * m * m, d), x_out=_bf16(g, B, N, o))
    t["idx"], t["nrec"], _ = _ids(g, B, N, c["reuse"])
    return t


# ---------------------------------------------------------------------------------------- run
def _sel(o):
    return dict(sim=o.sim, energy=o.energy, reuse_mask=o.reuse_mask, recompute_idx=o.recompute_idx,
                n_recompute=o.n_recompute, shift=o.shift, scalars=o.scalars, counts=o.counts, flags=o.flags)


def run(s):
    kind = s["case"]["kind"]
    if kind == "select":
        fc.fc_select(s["ctx"], s["prm"], s["prev"], s["cur"], s["out"][0])
        return _sel(s["out"][0])
    if kind == "carry":
        st = s["states"]
        fc.fc_select_carry(s["ctx"], s["prm"], st[0], s["cur"], st[1], s["out"][0])
        fc.fc_select_carry(s["ctx"], s["prm"], st[1], s["prev"], st[2], s["out"][1])
        return [_sel(s["out"][0]), _sel(s["out"][1])]
    if kind == "phase":
        fc.fc_phase_correlate(s["ctx"], s["prev"], s["cur"], s["shift_px"], s["peak"], s["resp"])
        return dict(shift_px=s["shift_px"], peak=s["peak"], response=s["resp"])
    if kind == "layer":
        fc.fc_layer_forward(s["ctx"], s["desc"], s["kv"], s["x"], s["idx"], s["nrec"], s["y"])
        return dict(y=s["y"], k=s["k"], v=s["v"])
    if kind == "trail":
        fc.fc_layer_forward_trail(s["ctx"], s["desc"], s["kv"], s["x"], s["y"])
        return dict(y=s["y"], k=s["k"], v=s["v"])
    if kind == "remap":
        fc.fc_cache_update_layers(s["ctx"], s["desc"], s["kvs"], s["yp"], s["yc"], s["shift"], s["mask"],
                                  s["case"]["grid_w"])
        last = s["kvs"][-1]
        first = s["kvs"][0]
        return dict(y=s["yc"], k=[first.k, last.k], v=[first.v, last.v])
    if kind == "vit":
        fc.fc_vit_block_forward(s["ctx"], s["desc"], s["cache"], s["x"], s["idx"], s["nrec"], s["y"])
        return dict(y=s["y"], k=s["k"], v=s["v"])
    if kind == "vitmap":
        fc.fc_vit_cache_update(s["ctx"], s["desc"], s["cache"], s["y_prev"], s["y"], s["shift"], s["mask"])
        return dict(y=s["y"], k=s["k"], v=s["v"])
    if kind == "merger":
        fc.fc_vit_merger_forward(s["ctx"], s["desc"], s["y"], s["idx"], s["nrec"], s["x_out"])
        return s["x_out"]
    o = s["sel"]
    fc.fc_select_carry(s["ctx"], s["prm"], s["states"][0], s["cur"], s["states"][1], o)
    x = s["emb"]
    for b in s["vit"]:
        fc.fc_vit_cache_update(s["ctx"], b["desc"], b["cache"], None, None, o.shift, o.reuse_mask)
        fc.fc_vit_block_forward(s["ctx"], b["desc"], b["cache"], x, o.recompute_idx, o.n_recompute, b["y"])
        x = b["y"]
    fc.fc_vit_merger_forward(s["ctx"], s["merger"], x, o.recompute_idx, o.n_recompute, s["x"])
    fc.fc_cache_update_layers(s["ctx"], s["lay"][0]["desc"], [b["kv"] for b in s["lay"]],
                              [b["yp"] for b in s["lay"]], [b["y"] for b in s["lay"]], o.shift,
                              o.reuse_mask, s["gw"])
    x = s["x"]
    for b in s["lay"]:
        fc.fc_layer_forward(s["ctx"], b["desc"], b["kv"], x, o.recompute_idx, o.n_recompute, b["y"])
        x = b["y"]
    return dict(sel=_sel(o), vit_y=[b["y"] for b in s["vit"]], x=s["x"], y=[b["y"] for b in s["lay"]],
                k=[b["k"] for b in s["lay"]], v=[b["v"] for b in s["lay"]])


# --------------------------------------------------------------------------------------- work
def _layer_work(shape, items, rows, tokens, window, text, trail):
    """rows: recomputed rows of all items."""
    d, nh, nkv, hd, f = LAYERS[shape]
    q = (nh + 2 * nkv) * hd
    S = text + window * tokens + trail
    weights = 2 * (q * d + q + d * nh * hd + 3 * f * d + 2 * d)
    cache = 2 * 2 * items * S * nkv * hd                 # every cached key and value read once
    acts = 2 * rows * (2 * d + 2 * nkv * hd)             # x in, y, k, v out
    keys = S - (trail or tokens) / 2                     # causal within the own region
    return (weights + cache + acts,
            2.0 * rows * (q * d + d * nh * hd + 3 * f * d) + 4.0 * rows * nh * hd * keys)


def _vit_work(shape, items, rows, patches, keys):
    d, H, hd, f = VITS[shape]
    f = 3420 if shape == "qwen" else f
    weights = 2 * (4 * d * d + 3 * f * d + 6 * d + 2 * f)
    acts = 2 * rows * (2 * d + 2 * d) + 2 * 2 * (items * patches - rows) * d
    return weights + acts, 2.0 * rows * (4 * d * d + 3 * f * d) + 4.0 * rows * d * keys


def _merger_work(shape, rows):
    d, m, o = MERGERS[shape]
    h = m * m * d
    return 2 * (h * h + h * o + h + o) + 2 * rows * (h + o), 2.0 * rows * (h * h + h * o)


def _select_work(items, h, w, merge, frames, align):
    n = (h // (P * merge)) * (w // (P * merge))
    b = items * (frames * 12 * h * w + n * (4 + 8 + 1 + 4 + 1))
    f = items * frames * h * w * (3 + 4.0 * P)            # luma and the patch transforms
    if align == "pixel":                                   # two forward transforms and one inverse
        f += items * 1.5 * 5 * h * w * math.log2(h * w)
    return b, f


def work(case):
    c, kind = case, case["kind"]
    if kind == "select":
        b, f = _select_work(c["items"], c["h"], c["w"], c["merge"], 2, c["align"])
    elif kind == "carry":   # two steps, each reads one frame and the spectra of the one before it
        b, f = _select_work(2 * c["items"], c["h"], c["w"], c["merge"], 1, "grid")
        b += 2 * 2 * c["items"] * 408 * (c["h"] // P) * (c["w"] // P)
    elif kind == "phase":
        hw = c["h"] * c["w"]
        b = c["items"] * (2 * 12 * hw + 8 * hw)
        f = c["items"] * (6 * hw + 1.5 * 5 * hw * math.log2(hw))
    elif kind in ("layer", "trail"):
        U = c.get("trail", 0)
        rows = c["items"] * U or sum(c["tokens"] - _reused(i, c["tokens"], c["reuse"])
                                     for i in range(c["items"]))
        b, f = _layer_work(c["shape"], c["items"], rows, c["tokens"], c["window"], c["text"], U)
    elif kind == "remap":
        d, nh, nkv, hd, _ = LAYERS[c["shape"]]
        rows = sum(_reused(i, c["tokens"], c["reuse"]) for i in range(c["items"]))
        b, f = 2 * c["layers"] * rows * 2 * (2 * nkv * hd + d), 0
    elif kind in ("vit", "vitmap"):
        N, mm = c["grid_h"] * c["grid_w"], c["merge"] ** 2
        reused = sum(_reused(i, N, c["reuse"]) for i in range(c["items"]))
        if kind == "vit":
            keys = mm * (min(c["window"], c["grid_h"]) * min(c["window"], c["grid_w"]) or N)
            b, f = _vit_work(c["shape"], c["items"], mm * (c["items"] * N - reused), N * mm, keys)
        else:
            b, f = 2 * 3 * 2 * max(1, mm * reused) * VITS[c["shape"]][0], 0
    elif kind == "merger":
        rows = sum(c["tokens"] - _reused(i, c["tokens"], c["reuse"]) for i in range(c["items"]))
        b, f = _merger_work(c["shape"], rows)
    else:                   # at the reuse that these frames give, about 37 %
        N = (c["h"] // 28) * (c["w"] // 28)
        n = N - 37 * N // 100
        b, f = _select_work(1, c["h"], c["w"], 2, 1, "grid")
        for keys in (min(64, 4 * N), 4 * N):
            vb, vf = _vit_work("qwen", 1, 4 * n, 4 * N, keys)
            b, f = b + vb + 2 * 2 * 2 * 4 * (N - n) * 1280, f + vf
        mb, mf = _merger_work("qwen", n)
        lb, lf = _layer_work("qwen", 1, n, N, c["window"], c["text"], 0)
        b, f = b + mb + 2 * lb + 2 * 2 * 2 * (N - n) * (1024 + 3584), f + mf + 2 * lf
    return {"bytes": int(b), "flops": float(f)}


# ---------------------------------------------------------------------------------- tolerance
def tolerance(case):
    kind = case["kind"]
    if kind in ("remap", "vitmap"):
        return "exact"                                  # rows are copied
    if kind in ("select", "carry"):
        return {"rel": 2e-6, "max": 2e-5}               # similarities are fp32 sums of 196 products
    if kind == "phase":
        return {"rel": 1e-9, "max": 1e-6}               # fp64 transforms of up to 896 x 448 points
    # bf16 operands and results: another order of the fp32 sums flips roundings of the stored
    # activations, one unit in 2^8 for a value that is rounded the other way
    if kind == "step":
        return {"rel": 1.2e-2, "max": 0.15}
    return {"rel": 6e-3, "max": 0.08}


# -------------------------------------------------------------------------------------- exact
def _f64(t):
    return t.to(torch.float64)


def _lin(x, w, b=None):
    y = x @ _f64(w).t().contiguous()
    return y if b is None else y + _f64(b)


def _norm(x, g):
    return x / torch.sqrt((x * x).mean(-1, keepdim=True) + 1e-6) * _f64(g)


def _rot(x, ang):
    """Rotate-half rotation of x [rows, heads, hd] by ang [rows, hd / 2]."""
    h = x.shape[-1] // 2
    cs, sn = torch.cos(ang)[:, None], torch.sin(ang)[:, None]
    return torch.cat([x[..., :h] * cs - x[..., h:] * sn, x[..., h:] * cs + x[..., :h] * sn], -1)


def _attend(q, k, v, see):
    """q [n, H, hd], k and v [S, Hkv, hd], see [n, S] -> [n, H hd]."""
    n, H, hd = q.shape
    out = torch.empty_like(q)
    for i in range(H):
        j = i // (H // k.shape[1])
        sc = q[:, i].contiguous() @ k[:, j].t().contiguous() / math.sqrt(hd)
        p = torch.softmax(sc.masked_fill(~see, -math.inf), -1)
        out[:, i] = p @ v[:, j].contiguous()
    return out.reshape(n, H * hd)


def _layer_angles(pos, hd, mrope, text, tokens, window, gw):
    """Rotation angles [rows, hd / 2] of the tokens at prompt indices pos."""
    inv = 1e6 ** (-2.0 * torch.arange(hd // 2, dtype=torch.float64, device=DEV) / hd)
    if not mrope:
        return pos[:, None].double() * inv
    span = max(tokens // gw, gw)
    r = pos - text
    frame, tok = r // tokens, r % tokens
    st = text + frame * span
    seen = (r >= 0) & (frame < window)
    late = r >= window * tokens
    plain = torch.where(late, pos - window * tokens + window * span, pos)
    p3 = [torch.where(seen, a, plain) for a in (st, st + tok // gw, st + tok % gw)]
    comp = torch.stack([p3[i] for i, n in enumerate(MROPE) for _ in range(n)], 1)
    return comp.double() * inv


def _layer_exact(shape, w, x, k, v, rows, qpos, kpos, angles):
    """Outputs of the rows x [n, d] (float64); k, v [S, Hkv, hd] float64 are written at rows."""
    d, nh, nkv, hd, f = LAYERS[shape]
    n = x.shape[0]
    qkv = _lin(_norm(x, w["g_attn"]), w["w_qkv"], w["b_qkv"])
    q, kn, vn = qkv.split([nh * hd, nkv * hd, nkv * hd], 1)
    k[rows], v[rows] = kn.reshape(n, nkv, hd), vn.reshape(n, nkv, hd)
    a = _attend(_rot(q.reshape(n, nh, hd), angles(qpos)), _rot(k, angles(kpos)), v,
                kpos[None] <= qpos[:, None])
    h1 = x + _lin(a, w["w_o"])
    h2 = _norm(h1, w["g_mlp"])
    return h1 + _lin(torch.nn.functional.silu(_lin(h2, w["w_gate"])) * _lin(h2, w["w_up"]), w["w_down"])


def _layout(text, tokens, window, trail):
    """Prompt index of every cache row (ring head window // 2) and the current frame's first row."""
    head = window // 2
    slot = torch.arange(window, device=DEV)
    first = text + ((slot - head) % window) * tokens
    frames = (first[:, None] + torch.arange(tokens, device=DEV)).reshape(-1)
    end = text + window * tokens
    kpos = torch.cat([torch.arange(text, device=DEV), frames, torch.arange(end, end + trail, device=DEV)])
    return kpos, text + ((head + window - 1) % window) * tokens


def _layer_case_exact(c, t):
    U, N = c.get("trail", 0), c["tokens"]
    hd = LAYERS[c["shape"]][3]
    kpos, cur0 = _layout(c["text"], N, c["window"], U)
    ang = lambda p: _layer_angles(p, hd, c["mrope"], c["text"], N, c["window"], c["grid_w"])  # noqa: E731
    k, v, y = _f64(t["k"]), _f64(t["v"]), _f64(t["y"])
    for b in range(c["items"]):
        if U:
            rows = torch.arange(t["S"] - U, t["S"], device=DEV)
            y[b] = _layer_exact(c["shape"], t["w"], _f64(t["x"][b]), k[b], v[b], rows, rows, kpos, ang)
        else:
            i = t["idx"][b, :int(t["nrec"][b])].long()
            qpos = c["text"] + (c["window"] - 1) * N + i
            y[b, i] = _layer_exact(c["shape"], t["w"], _f64(t["x"][b])[i], k[b], v[b], cur0 + i, qpos,
                                   kpos, ang)
    return dict(y=y, k=k, v=v)


def _vit_block_exact(shape, w, x, k, v, y, tokens, gh, gw, m, win):
    """One item: x, y [Np, d], k, v [Np, H, hd] float64; y, k and v are written at the tokens' patches."""
    d, H, hd, f = VITS[shape]
    mm = m * m
    Np = gh * gw * mm
    rows = (tokens[:, None] * mm + torch.arange(mm, device=DEV)).reshape(-1)
    p = torch.arange(Np, device=DEV)
    tok, sub = p // mm, p % mm
    pr, pc = (tok // gw) * m + sub // m, (tok % gw) * m + sub % m
    inv = 1e4 ** (-torch.arange(0, hd // 2, 2, dtype=torch.float64, device=DEV) / (hd // 2))
    ang = torch.cat([pr[:, None] * inv, pc[:, None] * inv], 1)
    wid = (tok // gw) // win * -(-gw // win) + (tok % gw) // win if win else torch.zeros_like(tok)
    xr = x[rows]
    n = rows.numel()
    q, kn, vn = _lin(_norm(xr, w["g1"]), w["w_qkv"], w["b_qkv"]).reshape(n, 3, H, hd).unbind(1)
    k[rows], v[rows] = kn, vn
    a = _attend(_rot(q, ang[rows]), _rot(k, ang), v, wid[rows][:, None] == wid[None])
    h1 = xr + _lin(a, w["w_o"], w["b_o"])
    gu = _lin(_norm(h1, w["g2"]), w["w_gate_up"], w["b_gate_up"])
    y[rows] = h1 + _lin(torch.nn.functional.silu(gu[:, :f]) * gu[:, f:], w["w_down"], w["b_down"])


def _merger_exact(w, y, tokens, m, d):
    """y [Np, d] float64 -> [len(tokens), d_out]."""
    rows = (tokens[:, None] * m * m + torch.arange(m * m, device=DEV)).reshape(-1)
    h = _norm(y[rows], w["g"]).reshape(tokens.numel(), m * m * d)
    return _lin(torch.nn.functional.gelu(_lin(h, w["w1"], w["b1"])), w["w2"], w["b2"])


def _luma(f):
    f = f.double()
    return 0.299 * f[:, 0] + 0.587 * f[:, 1] + 0.114 * f[:, 2]


def _phase(fp, fcur):
    """The phase-correlation surface of the spectra [B, h, w]."""
    x = fp * fcur.conj()
    mag = x.abs()
    keep = mag > 1e-9 * mag.amax((1, 2), keepdim=True)
    return torch.fft.ifft2(torch.where(keep, x / torch.where(keep, mag, torch.ones_like(mag)),
                                       torch.zeros_like(x))).real


def _signed(i, n):
    return torch.where(i <= n // 2, i, i - n)


def _pixel_shift(yp, yc):
    """Sub-pixel displacement [B, 2], integer peak and surface of full-resolution luma."""
    B, h, w = yp.shape
    r = _phase(torch.fft.fft2(yp), torch.fft.fft2(yc))
    at = r.reshape(B, -1).argmax(1)
    i, j, b = at // w, at % w, torch.arange(B, device=DEV)

    def vertex(a, m, z):
        den = a - 2 * m + z
        return torch.where(den >= 0, torch.zeros_like(den), (a - z) / (2 * den))
    mid = r[b, i, j]
    di = _signed(i, h) + vertex(r[b, (i - 1) % h, j], mid, r[b, (i + 1) % h, j])
    dj = _signed(j, w) + vertex(r[b, i, (j - 1) % w], mid, r[b, i, (j + 1) % w])
    return torch.stack([di, dj], 1), r


def _select_exact(prev, cur, m, align="grid", adaptive=True):
    """Algorithm 1 at the paper's parameters (tau_mig 0.12, lambda 0.25, reuse between 8 % and 50 %)."""
    B, _, h, w = cur.shape
    ph, pw = h // P, w // P
    gh, gw = ph // m, pw // m
    M = gh * gw
    yc, yp = _luma(cur), _luma(prev)

    def tiles(y):
        return y.reshape(B, ph, P, pw, P).transpose(2, 3)

    def tokens(a):     # [B, ph, pw, ...] -> [B, gh, gw, m * m, ...]
        a = a.reshape(B, gh, m, gw, m, *a.shape[3:])
        return a.transpose(2, 3).reshape(B, gh, gw, m * m, *a.shape[5:])
    tc, tp = tiles(yc), tiles(yp)
    ac, ap = (tokens(torch.fft.fft2(t).abs()).reshape(B, gh, gw, -1) for t in (tc, tp))
    fcur, fprev = (torch.fft.fft2(tokens(t.mean((-1, -2))).mean(-1)) for t in (tc, tp))
    k = torch.arange(P, dtype=torch.float64, device=DEV)
    dct = torch.cos(math.pi * (2 * k[None] + 1) * k[:, None] / (2 * P)) * math.sqrt(2 / P)
    dct[0] = math.sqrt(1 / P)
    coef = dct @ tc @ dct.t()
    coef[..., :3, :3] = 0
    e = tokens(coef.square().sum((-1, -2))).sum(-1).reshape(B, M)
    e = torch.where(e < 1e-8 * m * m, torch.zeros_like(e), e)
    a, b = fcur.abs(), fprev.abs()
    na, nb = a.square().sum((1, 2)).sqrt(), b.square().sum((1, 2)).sqrt()
    simf = (a * b).sum((1, 2)) / (na * nb)
    pr = a.square().reshape(B, M) / na.square()[:, None]
    psi = -torch.where(pr > 0, pr * pr.clamp_min(1e-300).log(), torch.zeros_like(pr)).sum(1) / math.log(M)
    alpha = 0.08 + 0.42 * torch.exp(-psi) if adaptive else torch.full_like(psi, 0.5)
    if align == "pixel":
        d = _pixel_shift(yp, yc)[0]
        shift = (torch.sign(d) * torch.floor(d.abs() / (P * m) + 0.5)).long()
    else:
        at = _phase(fprev, fcur).reshape(B, M).argmax(1)
        shift = torch.stack([_signed(at // gw, gh), _signed(at % gw, gw)], 1)
    i = torch.arange(gh, device=DEV).view(1, gh, 1) + shift[:, 0].view(B, 1, 1)
    j = torch.arange(gw, device=DEV).view(1, 1, gw) + shift[:, 1].view(B, 1, 1)
    ok = (i >= 0) & (i < gh) & (j >= 0) & (j < gw)
    src = (i.clamp(0, gh - 1) * gw + j.clamp(0, gw - 1)).reshape(B, M)
    al = ok.reshape(B, M)
    u = ac.reshape(B, M, -1)
    v = ap.reshape(B, M, -1).gather(1, src[..., None].expand(B, M, u.shape[-1]))
    sim = torch.where(al, (u * v).sum(-1) / (u.norm(dim=-1) * v.norm(dim=-1)), torch.zeros_like(e))
    mu, sd = e.mean(1), e.std(1, unbiased=False)
    thr = mu + 0.25 * sd
    cand = al & ~(e > thr[:, None])
    budget = torch.floor(alpha * M).long()
    final = torch.where(simf < 0.12, torch.zeros_like(budget), torch.minimum(budget, cand.sum(1)))
    order = torch.where(cand, e, torch.full_like(e, math.inf)).argsort(dim=1, stable=True)
    rank = torch.empty_like(order).scatter_(1, order, torch.arange(M, device=DEV).expand(B, M))
    reuse = rank < final[:, None]
    scalars = torch.stack([simf, psi, alpha, mu, sd, thr], 1)
    return dict(sim=sim, energy=e, scalars=scalars, reuse=reuse, shift=shift)


_WHOLE = dict.fromkeys(("reuse_mask", "recompute_idx", "n_recompute", "shift", "counts", "flags"))


def _sel_exact(*a, **kw):
    r = _select_exact(*a, **kw)
    return dict(_WHOLE, sim=r["sim"], energy=r["energy"], scalars=r["scalars"])


def _remapped(dst, src, shift, reuse, gh, gw):
    """dst [N, ...] with the rows of src [N, ...] at each reused token's source."""
    t = reuse.nonzero()[:, 0]
    s = (t // gw + shift[0]) * gw + t % gw + shift[1]
    out = dst.clone()
    out[t] = src[s]
    return out


def exact(case, seed):
    c, g = case, _gen(seed)
    kind = c["kind"]
    if kind in ("select", "carry", "phase"):
        prev, cur = _frames(g, c["items"], c["h"], c["w"])
        if kind == "select":
            return _sel_exact(prev, cur, c["merge"], c["align"], c["adaptive"])
        if kind == "carry":
            return [_sel_exact(prev, cur, c["merge"]), _sel_exact(cur, prev, c["merge"])]
        d, r = _pixel_shift(_luma(prev), _luma(cur))
        return dict(shift_px=d, peak=None, response=r)
    if kind in ("layer", "trail"):
        return _layer_case_exact(c, _layer_inputs(c, g))
    if kind == "vit":
        t = _vit_inputs(c, g)
        k, v, y = _f64(t["k"]), _f64(t["v"]), _f64(t["y"])
        for b in range(c["items"]):
            _vit_block_exact(c["shape"], t["w"], _f64(t["x"][b]), k[b], v[b], y[b],
                             t["idx"][b, :int(t["nrec"][b])].long(), c["grid_h"], c["grid_w"], c["merge"],
                             c["window"])
        return dict(y=y, k=k, v=v)
    if kind == "merger":
        d, m, o = MERGERS[c["shape"]]
        t = _merger_inputs(c, g)
        x = _f64(t["x_out"])
        for b in range(c["items"]):
            i = t["idx"][b, :int(t["nrec"][b])].long()
            x[b, i] = _merger_exact(t["w"], _f64(t["y"][b]), i, m, d)
        return x
    if kind in ("remap", "vitmap"):
        return None                                     # copies: "exact" says it all
    t = _step_inputs(c, g)
    gh, gw, N = t["gh"], t["gw"], t["N"]
    hd = LAYERS["qwen"][3]
    r = _select_exact(t["prev"], t["cur"], 2)
    reuse, shift = r["reuse"][0], r["shift"][0]
    i = (~reuse).nonzero()[:, 0]
    x, vit_y = _f64(t["emb"][0]), []
    for b in t["vit"]:
        k, v = (_remapped(_f64(b[n][0]).reshape(N, 4, 16, 80), _f64(b[n + "p"][0]).reshape(N, 4, 16, 80),
                          shift, reuse, gh, gw).reshape(4 * N, 16, 80) for n in ("k", "v"))
        y = _f64(b["y"][0])
        _vit_block_exact("qwen", b["w"], x, k, v, y, i, gh, gw, 2, b["win"])
        vit_y.append(y[None])
        x = y
    xm = _f64(t["x"][0])
    xm[i] = _merger_exact(t["mw"], x, i, 2, 1280)
    kpos, cur0 = _layout(c["text"], N, c["window"], 0)
    head = c["window"] // 2
    prev0 = c["text"] + ((head + c["window"] - 2) % c["window"]) * N
    ang = lambda p: _layer_angles(p, hd, True, c["text"], N, c["window"], gw)  # noqa: E731
    x, out = xm, dict(y=[], k=[], v=[])
    for b in t["lay"]:
        k, v = _f64(b["k"][0]), _f64(b["v"][0])
        for a in (k, v):
            a[cur0:cur0 + N] = _remapped(a[cur0:cur0 + N], a[prev0:prev0 + N].clone(), shift, reuse, gh, gw)
        y = _remapped(_f64(b["y"][0]), _f64(b["yp"][0]), shift, reuse, gh, gw)
        y[i] = _layer_exact("qwen", b["w"], x[i], k, v, cur0 + i, c["text"] + (c["window"] - 1) * N + i,
                            kpos, ang)
        for n, a in (("y", y), ("k", k), ("v", v)):
            out[n].append(a[None])
        x = y
    sel = dict(_WHOLE, sim=r["sim"], energy=r["energy"], scalars=r["scalars"])
    return dict(sel=sel, vit_y=vit_y, x=xm[None], **out)
