"""The work a user of this framework has it do: decoding records of progressive JPEG images at a chosen scan group,
raising a batch's fidelity, feeding a training loop from host memory, scoring fidelity, and making records.

Sizes follow the workloads of pcrgen (64 x 64 gray, 256 x 256, photographs of 300 to 500 pixels, 1024 x 1024, 600 x 450
in 4:4:4) and the spread of image sizes in between.  A case is a dict of plain values:

  op        decode    every record of the batch to uint8 pixels, one handle and one stream per record
            upgrade   one record at scan group k0, then raised to k
            crop      decode and training tail (random boxes to `out` x `out` half-precision tensors), records resident
            load      the same from pinned host memory through the loader: copy, bind, decode, tail
            score     MS-SSIM of the pictures at scan group k against those of the last one
            encode    baseline files to a record of progressive files (decode, count, transcode, group, index)
  mode      decode only: replicate / triangle / smooth (up-sampling of chroma, smoothing of DC-only components)
  records, images (per record), w0..w1, h0..h1 (sides drawn uniformly), channels, sub (chroma sub-sampling)
  quality, sigma (noise; each picture has its own strength around it), restart (MCU rows per restart interval, 0: none)
  entry     MCUs between entry points (0: a plain record)
  k, k0, out
"""
import math
import os
from concurrent.futures import ThreadPoolExecutor

import numpy as np
import torch

import paper_1911_00472_amd as pcr
import pcrgen

MEAN, INV_STD = (0.485, 0.456, 0.406), (1 / 0.229, 1 / 0.224, 1 / 0.225)
DISTINCT_PIXELS = 16 << 20                  # of a batch's pictures about this many pixels are different ones


def _case(name, op, records, images, size, k, channels=3, sub=2, quality=90, sigma=26.0, restart=0, entry=64, mode="replicate", k0=0, out=0):
    return {"name": name, "op": op, "mode": mode, "records": records, "images": images, "w0": size[0], "w1": size[1], "h0": size[2], "h1": size[3],
            "channels": channels, "sub": sub, "quality": quality, "sigma": sigma, "restart": restart, "entry": entry, "k": k, "k0": k0, "out": out}


PHOTO = (300, 500, 300, 500)


def listed():
    return [
        # a handful of gray thumbnails from a plain record: launches and latency
        _case("gray64_k6", "decode", 1, 64, (64, 64, 64, 64), 6, channels=1, sub=1, sigma=8.0, entry=0),
        # small pictures of every size and shape, as crawled data holds them
        _case("ragged_k10", "decode", 1, 256, (17, 320, 17, 320), 10, sigma=16.0),
        # one record of a small-image dataset at half fidelity
        _case("rgb256_k5", "decode", 1, 1024, (256, 256, 256, 256), 5, sigma=9.0),
        # a shuffled epoch over photographs, four records in flight: lowest and full fidelity
        _case("photo_k1", "decode", 4, 1024, PHOTO, 1),
        _case("photo_k10", "decode", 4, 1024, PHOTO, 10),
        # a record another tool grouped, without entry points
        _case("photo_plain_k10", "decode", 1, 512, PHOTO, 10, entry=0),
        # high-resolution pictures with restart markers, half fidelity
        _case("hires_k5", "decode", 2, 128, (1024, 1024, 1024, 1024), 5, sigma=9.0, restart=1, entry=0),
        # dermatology-like pictures: full chroma, high quality
        _case("ham444_k10", "decode", 1, 256, (600, 600, 450, 450), 10, sub=1, quality=95, sigma=18.0),
        # a loss plateau: the batch decoded at a low fidelity is raised to the full one
        _case("upgrade_2_10", "upgrade", 1, 1024, PHOTO, 10, k0=2),
        # training input from storage buffers: 224 x 224 crops at the fidelity the paper trains at
        _case("load_crop_k5", "load", 4, 512, PHOTO, 5, out=224),
        # which scan group is good enough: MS-SSIM of a record
        _case("score_k2", "score", 1, 1024, PHOTO, 2),
        # making a dataset: baseline files into an indexed record
        _case("encode_64", "encode", 1, 64, PHOTO, 10),
    ]


def draw(rng):
    op = rng.choices(["decode", "upgrade", "crop", "load", "score", "encode"], [60, 8, 8, 8, 8, 8])[0]
    channels = rng.choices([3, 1], [85, 15])[0]
    sub = 1 if channels == 1 or rng.random() < 0.2 else 2
    last = 10 if channels == 3 else 6
    side = math.exp(rng.uniform(math.log(24), math.log(1024)))
    w = max(9, round(side * rng.uniform(0.75, 1.33)))
    h = max(9, round(side * side / w))
    spread = rng.choice([1.0, 1.0, 1.6])
    records = 1 if op in ("upgrade", "score", "encode") else rng.choice([1, 1, 2, 4])
    most = {"encode": 1e7, "score": 1.2e8, "load": 1.2e8}.get(op, 2.5e8)         # pixels of the batch
    pixels = math.exp(rng.uniform(math.log(2.6e5), math.log(most)))
    images = min(2048, max(1, int(pixels / records / (w * h))))
    restart = 1 if op != "encode" and rng.random() < 0.15 else 0
    entry = 0 if restart or (op != "encode" and rng.random() < 0.25) else rng.choice([32, 64, 64, 100, 128])
    k = last if op == "encode" else rng.randint(1, last)
    k0 = 0
    if op == "upgrade":
        k = rng.randint(2, last)
        k0 = rng.randint(1, k - 1)
    mode = rng.choices(["replicate", "triangle", "smooth"], [85, 8, 7])[0] if op == "decode" else "replicate"
    c = _case("", op, records, images, (int(w / spread), int(w * spread), int(h / spread), int(h * spread)), k, channels=channels, sub=sub,
              quality=rng.randint(75, 95), sigma=round(rng.uniform(3, 30), 1), restart=restart, entry=entry, mode=mode, k0=k0,
              out=rng.choice([96, 160, 224]) if op in ("crop", "load") else 0)
    del c["name"]
    return c


# ---- inputs ----

def _pictures(case, count, gen):
    """[count, channels, h1, w1] float32 pictures 0..255 on the GPU: octaves of value noise, rectangles, noise."""
    C, H, W = case["channels"], -(-case["h1"] // 16) * 16, -(-case["w1"] // 16) * 16
    dev = gen.device

    def rand(*shape):
        return torch.rand(shape, generator=gen, device=dev)

    x = torch.full((count, C, H, W), 128.0, device=dev)
    for cell in (128, 64, 32, 16, 8, 4):
        gh, gw = H // cell + 2, W // cell + 2
        coarse = (rand(count, 1, gh, gw) - 0.5) + 0.5 * (rand(count, C, gh, gw) - 0.5)
        fine = torch.nn.functional.interpolate(coarse, size=(gh * cell, gw * cell), mode="bilinear", align_corners=False)
        x += (4.5 * cell ** 0.6) * fine[:, :, cell // 2:cell // 2 + H, cell // 2:cell // 2 + W]
    yy, xx = torch.arange(H, device=dev).view(1, 1, H, 1), torch.arange(W, device=dev).view(1, 1, 1, W)
    for _ in range(5):
        y0, x0 = (rand(count, 1, 1, 1) * H).int(), (rand(count, 1, 1, 1) * W).int()
        h, w = (rand(count, 1, 1, 1) * H / 3).int(), (rand(count, 1, 1, 1) * W / 3).int()
        inside = (yy >= y0) & (yy < y0 + h) & (xx >= x0) & (xx < x0 + w)
        x += inside * (rand(count, C, 1, 1) - 0.5) * 120
    strength = case["sigma"] * (0.25 + 1.5 * rand(count, 1, 1, 1))
    x += strength * torch.randn((count, C, H, W), generator=gen, device=dev)
    return x.clamp_(0, 255).round_()


def _coefficients(case, x):
    """Quantised coefficient planes of the pictures: int16 [count, rows, columns, 64] per component, on the host; the tables."""
    tables = pcrgen.quant_tables(case["quality"])
    i = torch.arange(8, dtype=torch.float64)
    zz = sorted(range(64), key=lambda p: (p // 8 + p % 8, (p // 8 if (p // 8 + p % 8) % 2 else p % 8)))
    basis = torch.cos((2 * i[None, :] + 1) * i[:, None] * math.pi / 16) / 2
    basis[0] /= math.sqrt(2.0)
    basis = basis.float().to(x.device)
    if x.shape[1] == 3:
        r, g, b = x[:, 0], x[:, 1], x[:, 2]
        planes = [0.299 * r + 0.587 * g + 0.114 * b, 128 - 0.168736 * r - 0.331264 * g + 0.5 * b, 128 + 0.5 * r - 0.418688 * g - 0.081312 * b]
        if case["sub"] == 2:
            planes[1:] = [torch.nn.functional.avg_pool2d(p[:, None], 2)[:, 0] for p in planes[1:]]
    else:
        planes = [x[:, 0]]
    out = []
    for c, p in enumerate(planes):
        q = torch.empty(64)
        q[torch.tensor(zz)] = torch.from_numpy(tables[min(c, 1)].astype(np.float32))
        n, h, w = p.shape
        v = (p - 128).reshape(n, h // 8, 8, w // 8, 8).transpose(2, 3).reshape(-1, 8, 8)
        v = (v.reshape(-1, 8) @ basis.t()).reshape(-1, 8, 8).transpose(1, 2).contiguous()       # [block, frequency x, y]
        v = (v.reshape(-1, 8) @ basis.t()).reshape(-1, 8, 8).transpose(1, 2)                    # [block, frequency y, x]
        v = torch.round(v.reshape(-1, 64) / q.to(x.device)).clamp_(-1023, 1023)
        out.append(v.to(torch.int16).reshape(n, h // 8, w // 8, 64).cpu().numpy())
    return out, tables


def _files(case, seed, script=None):
    """(the JPEG files of every record, widths, heights), as a dataset on disk would hold them."""
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    rng = np.random.default_rng(191100472)              # the sizes belong to the case, what the pictures show to the seed
    total = case["records"] * case["images"]
    distinct = max(1, min(total, DISTINCT_PIXELS // (case["w1"] * case["h1"])))
    W, H = (rng.integers(case[a], case[b] + 1, size=distinct) for a, b in (("w0", "w1"), ("h0", "h1")))
    C, s = case["channels"], case["sub"]
    planes, tables = _coefficients(case, _pictures(case, distinct, gen))

    def one(i):
        mx, my = -(-int(W[i]) // (8 * s)), -(-int(H[i]) // (8 * s))
        parts = [p[i, :my * (s if c == 0 else 1), :mx * (s if c == 0 else 1)].reshape(-1) for c, p in enumerate(planes)]
        return pcrgen.encode_coefs(np.concatenate(parts), int(W[i]), int(H[i]), C, s, s, tables, script, case["restart"])

    pcrgen.lib()
    with ThreadPoolExecutor(min(16, os.cpu_count() or 1)) as ex:
        files = list(ex.map(one, range(distinct)))
    order = np.concatenate([rng.permutation(distinct) for _ in range(-(-total // distinct))])[:total]
    n = case["images"]
    return [[files[j] for j in order[a:a + n]] for a in range(0, total, n)], W[order], H[order]


def _record(case, files):
    return pcr.record_write_indexed(files, None, case["entry"]) if case["entry"] else pcr.record_write(files)


def _boxes(seed, W, H):
    """Random-resized-crop boxes: 8 to 100 % of the area, half of them mirrored; int32 [n, 5] on the GPU."""
    rng = np.random.default_rng(seed + 1)
    n = len(W)
    side = np.sqrt(rng.uniform(0.08, 1.0, n))
    ratio = np.exp(rng.uniform(math.log(3 / 4), math.log(4 / 3), n) / 2)
    w, h = (np.clip(np.rint(d * side * r), 1, d).astype(np.int64) for d, r in ((W, ratio), (H, 1 / ratio)))
    x, y = (np.floor(rng.uniform(0, 1, n) * (d - e + 1)).astype(np.int64) for d, e in ((W, w), (H, h)))
    return torch.from_numpy(np.stack([x, y, w, h, rng.integers(0, 2, n)], 1).astype(np.int32)).cuda()


class State:
    pass


def prepare(case, seed):
    S = State()
    S.case = case
    op, n = case["op"], case["images"]
    if op == "encode":                                                     # the files a dataset consists of
        files, W, H = _files(case, seed, "sequential")
        S.files = files[0]
        S.out = np.zeros(65536 + 2 * int((W * H).sum()), np.uint8)
        return S
    files, W, H = _files(case, seed)
    data = [_record(case, f) for f in files]
    S.outs, S.status = [], [torch.empty(n, dtype=torch.int32, device="cuda") for _ in data]
    if op in ("crop", "load"):
        S.boxes = [_boxes(seed + a, W[a:a + n], H[a:a + n]) for a in range(0, len(W), n)]
        S.outs = [torch.empty((n, case["channels"], case["out"], case["out"]), dtype=torch.float16, device="cuda") for _ in data]
    if op == "load":                                                       # prefixes as a reader has put them into the staging buffers
        S.sizes = []
        for d in data:
            ok, need = pcr.prefix_length(d[:24 + 8 * 16], case["k"])
            assert ok
            S.sizes.append(need)
        S.loader = pcr.Loader(len(data), max(S.sizes))
        for slot, d in enumerate(data):
            S.loader.staging(slot)[:S.sizes[slot]] = np.frombuffer(d, np.uint8, S.sizes[slot])
        S.streams = [torch.cuda.ExternalStream(S.loader.stream(slot)) for slot in range(len(data))]
        return S
    S.records = [pcr.pcr_open(d, 0) for d in data]
    S.streams = [torch.cuda.Stream() for _ in data]
    if op != "crop":
        S.outs = [torch.empty(int(r.output_layout()[-1]), dtype=torch.uint8, device="cuda") for r in S.records]
    if op == "score":
        r = S.records[0]
        S.top = r.decode_batch(r.G)
        r.decode_batch(case["k"], S.outs[0])
        S.scores = torch.empty(n, dtype=torch.float32, device="cuda")
    return S


def run(S):
    case = S.case
    op, k = case["op"], case["k"]
    if op == "encode":
        progressive = pcr.transcode_files(S.files)
        record = pcr.record_write_indexed(progressive, None, case["entry"])
        S.out[:len(record)] = np.frombuffer(record, np.uint8)
        return S.out, len(record)
    if op == "score":
        return S.records[0].msssim_batch(S.outs[0], S.top, S.scores)
    if op == "upgrade":
        r = S.records[0]
        r.decode_batch(case["k0"], S.outs[0], S.status[0])
        return r.upgrade_batch(k, S.outs[0], S.status[0]), S.status[0]
    here = torch.cuda.current_stream()
    for j, s in enumerate(S.streams):
        s.wait_stream(here)
        if op == "load":
            S.loader.upload(j, S.sizes[j])
            S.loader.decode_crop(j, k, S.boxes[j], case["out"], case["out"], MEAN, INV_STD, None, S.outs[j], S.status[j])
            continue
        r = S.records[j]
        if op == "crop":
            r.decode_crop_batch(k, S.boxes[j], case["out"], case["out"], MEAN, INV_STD, None, S.outs[j], S.status[j], s.cuda_stream)
        else:
            call = {"replicate": r.decode_batch, "triangle": r.decode_batch_triangle, "smooth": r.decode_batch_smooth}[case["mode"]]
            call(k, S.outs[j], S.status[j], s.cuda_stream)
    for s in S.streams:
        here.wait_stream(s)
    return S.outs, S.status


# share of a file that its first k scans take (the usual 10-scan and 6-scan scripts)
SHARE = {3: (0.05, 0.13, 0.15, 0.17, 0.3, 0.48, 0.49, 0.54, 0.59, 1.0), 1: (0.07, 0.17, 0.33, 0.56, 0.57, 1.0)}


def work(case):
    """Compressed bytes read once (from the bits a sample of such a picture takes at its noise and quality), outputs written
    once; operations: an inverse transform of 8 x 8 blocks (11 per sample), colour (9 per pixel)."""
    pixels = case["records"] * case["images"] * (case["w0"] + case["w1"]) * (case["h0"] + case["h1"]) / 4
    C = case["channels"]
    samples = pixels * (1 if C == 1 else 3 if case["sub"] == 1 else 1.5)
    bits = samples * min(6.0, 0.3 + 0.115 * case["sigma"] * 2.0 ** ((case["quality"] - 90) / 10))
    share = SHARE[C][min(case["k"], len(SHARE[C])) - 1]
    flops = 11 * samples + (9 * pixels if C == 3 else 0)
    op = case["op"]
    if op == "encode":                        # files in, record out
        return {"bytes": 2 * bits / 8, "flops": flops}
    if op == "score":                         # two pictures in; eleven-tap windows both ways over five products of every luma sample
        return {"bytes": 2 * C * pixels, "flops": 4 / 3 * pixels * 5 * 2 * 2 * 11}
    if op == "upgrade":                       # pixels at both fidelities
        return {"bytes": share * bits / 8 + 2 * C * pixels, "flops": 2 * flops}
    if op in ("crop", "load"):
        out = case["records"] * case["images"] * C * case["out"] ** 2
        return {"bytes": share * bits / 8 + 2 * out, "flops": flops + 8 * out}
    return {"bytes": share * bits / 8 + C * pixels, "flops": flops}


def tolerance(case):
    op = case["op"]
    if op == "encode":
        return "exact"
    if op == "score":                         # single-precision moments of 8-bit samples, a product of five powers
        return {"rel": 5e-5, "max": 3e-4}
    if op in ("crop", "load"):                # half precision; a source pixel may round to the next level
        return {"rel": 1e-3, "max": 0.02}
    return {"rel": 0.0, "differ": 5e-4}       # pixels whose single-precision value lies on the edge of rounding
