"""The workloads this framework's speed is judged on, each through its public entry points.

A case is a dict of plain values.  Its ``path`` says which part of the framework it calls:

* ``block``  -- one SPVConv block in one call: voxelize, kernel map, convs, devoxelize + point MLP;
* ``net``    -- the forward of the SPVCNN-style network: per-point logits;
* ``maps``   -- what a network's plan needs of the points: voxels, neighbour tables, stride-2 maps,
  child tables (and, for training, the submanifold pairs);
* ``conv``   -- one 3x3x3 layer of a network (conv + BN + residual + ReLU) on its stride's table;
* ``updown`` -- a stage change: the 2x2x2 stride-2 conv and the transposed one back;
* ``train_conv``  -- a training step of a 3x3x3 conv + BN + ReLU layer, forward and backward;
* ``train_point`` -- a training step of a point module: scatter-mean onto the stride's voxels,
  devoxelization, point MLP and fusion, forward and backward.

In the training steps the layer's raw product, which the backward of BN + ReLU reads, is given with
the other inputs and not taken from the forward call, so that no ReLU at the edge of zero turns on
the rounding of a sum.

Every cloud is made of seeded synthetic 64-beam sweeps (``synth.lidar_sweep``), each cut to a
sector of consecutive azimuths that holds the wanted number of points; ``scene`` picks the sweeps,
and batches of sweeps carry their batch index.  Features are N(0, 1) and weights have fan-in scaling.
"""
import functools
import math

import numpy as np
import torch

from paper_2007_16100_amd import spv, synth

DTYPES = {"f32": torch.float32, "bf16": torch.bfloat16, "f16": torch.float16}
CONV_WIDTHS = (32, 64, 96, 128, 256)  # the widths of the neighbour-table conv
SWEEP_POINTS = 120_000                # about a whole sweep

# voxels per point of a sweep at strides 1, 2, 4, 8, 16 of 0.05 m, and pairs per voxel of a 3x3x3 map
VOXELS = (0.70, 0.40, 0.14, 0.056, 0.023)
PAIRS = (6.6, 8.0, 9.5, 10.5, 11.0)


def listed():
    return [
        # a handful of points around one object, single precision: launches and latency
        dict(name="block_object_f32", path="block", scene=1, sweeps=1, points=2000, voxel=0.1, channels=16,
             dtype="f32", residual=False),
        # a cropped region of interest
        dict(name="block_crop_bf16", path="block", scene=2, sweeps=1, points=17001, voxel=0.05, channels=32,
             dtype="bf16", residual=False),
        # the block on one sweep at the paper's width: the headline workload
        dict(name="block_sweep_bf16", path="block", scene=3, sweeps=1, points=120000, voxel=0.05, channels=96,
             dtype="bf16", residual=False),
        # a batch, residual form, in half precision
        dict(name="block_batch_f16", path="block", scene=4, sweeps=3, points=300007, voxel=0.05, channels=64,
             dtype="f16", residual=True),
        # segmentation of one scan as a vehicle would run it, and of a batch as an evaluation would
        dict(name="net_sweep", path="net", scene=5, sweeps=1, points=110000, voxel=0.05, dtype="bf16"),
        dict(name="net_batch4", path="net", scene=6, sweeps=4, points=440000, voxel=0.05, dtype="bf16"),
        # the maps of a network on a batch, with the pairs that training needs
        dict(name="maps_batch2", path="maps", scene=7, sweeps=2, points=200003, voxel=0.05, pairs=True),
        # the decoder's widest full-resolution layer, and a deep layer at stride 8
        dict(name="conv_96_stride1", path="conv", scene=8, sweeps=4, points=440000, stride=0, cin=96, cout=96,
             dtype="bf16", residual=True),
        dict(name="conv_256_stride8", path="conv", scene=9, sweeps=4, points=440000, stride=3, cin=256, cout=256,
             dtype="bf16", residual=True),
        # a change of resolution, down and back up
        dict(name="updown_64_128", path="updown", scene=10, sweeps=1, points=120000, stride=0, fine=64, coarse=128,
             dtype="bf16"),
        # training steps of a conv layer and of a point module
        dict(name="train_conv_96", path="train_conv", scene=11, sweeps=1, points=120000, stride=0, cin=96, cout=96,
             dtype="bf16"),
        dict(name="train_point_96", path="train_point", scene=12, sweeps=1, points=120000, stride=2, channels=96,
             dtype="bf16"),
    ]


def draw(rng):
    def points(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    path = rng.choice(("block", "block", "net", "maps", "conv", "conv", "updown", "train_conv", "train_point"))
    n = points({"block": 1500, "net": 20000}.get(path, 10000), 440000)
    case = dict(path=path, scene=rng.randint(100, 999), sweeps=max(rng.choice((1, 2, 4)), -(-n // SWEEP_POINTS)),
                points=n)
    half = rng.choice(("bf16", "bf16", "f16"))
    if path == "block":
        dtype = rng.choice(("bf16", "bf16", "f16", "f32"))
        # the vector-ALU path of single precision is drawn at the sizes it is used at
        if dtype == "f32":
            case["points"] = n = min(n, points(1500, 60000))
        case.update(voxel=rng.choice((0.05, 0.05, 0.1)), channels=rng.choice((16, 32, 48) if dtype == "f32" else
                                                                            (16, 32, 48, 64, 96, 128)),
                    dtype=dtype, residual=rng.random() < 0.4)
    elif path == "net":
        case.update(voxel=0.05, dtype="bf16")
    elif path == "maps":
        case.update(voxel=0.05, pairs=rng.random() < 0.5)
    elif path in ("conv", "train_conv"):
        stride = rng.randint(0, 4 if path == "conv" else 2)
        # a network's widths grow with the stride
        widths = CONV_WIDTHS[:4] if stride < 2 else CONV_WIDTHS[1:]
        case.update(stride=stride, cin=rng.choice(widths), cout=rng.choice(widths), dtype=half)
        if path == "conv":
            case.update(residual=rng.random() < 0.5)
    elif path == "updown":
        case.update(stride=rng.randint(0, 3), fine=rng.choice((32, 64, 96, 128)), coarse=rng.choice((64, 96, 128)),
                    dtype=half)
    else:
        case.update(stride=rng.randint(0, 4), channels=rng.choice((32, 64, 96, 128)), dtype=half)
    case["sweeps"] = max(case["sweeps"], -(-n // SWEEP_POINTS))
    return case


# -- inputs ------------------------------------------------------------------

@functools.lru_cache(64)  # ray casting on the host: half a second a sweep
def sweep(seed):
    return synth.lidar_sweep(seed).astype(np.float64)


def cloud(case, seed):
    """The case's points [n][3] float32 and their batch index [n] int32 (None for one sweep).

    The scene gives the voxels; the seed turns, mirrors and shifts each sweep by whole voxels (of
    every stride) and places the points anew inside their voxels, so that another seed gives other
    points, another order of the voxels and other maps, but as many voxels at every stride."""
    rng = np.random.default_rng(int(seed))
    parts, batch, v = [], [], case.get("voxel", 0.05)
    for i in range(case["sweeps"]):
        want = (case["points"] + case["sweeps"] - 1 - i) // case["sweeps"]
        xyz = sweep(1000 * case["scene"] + i)
        turn = np.argsort(np.arctan2(xyz[:, 1], xyz[:, 0]), kind="stable")
        q = np.floor(xyz[np.sort(turn[:want])] / v)  # a sector, in the sensor's own order
        for _ in range(rng.integers(4)):
            q[:, 0], q[:, 1] = -1 - q[:, 1], q[:, 0].copy()
        if rng.integers(2):
            q[:, 1] = -1 - q[:, 1]
        q += 16 * rng.integers(-4, 5, size=3)
        parts.append(((q + rng.uniform(0.02, 0.98, size=q.shape)) * v).astype(np.float32))
        batch.append(np.full(len(q), i, np.int32))
    return np.concatenate(parts), np.concatenate(batch) if case["sweeps"] > 1 else None


class Draws:
    """Seeded values on the GPU."""

    def __init__(self, seed):
        self.gen = torch.Generator(device="cuda")
        self.gen.manual_seed(int(seed) * 1_000_003 + 17)

    def normal(self, *shape, std=1.0, dtype=torch.float32):
        return (torch.randn(*shape, generator=self.gen, device="cuda") * std).to(dtype)

    def bn(self, c):
        return torch.rand(c, generator=self.gen, device="cuda") + 0.5, self.normal(c, std=0.1)

    def weight(self, *shape, dtype):
        return self.normal(*shape, std=1.0 / math.sqrt(math.prod(shape[:-1])), dtype=dtype)


def layers():
    """(name, shape, with BN) of every layer of the network, in order."""
    w = synth.SPVCNN_WIDTHS
    out = [("stem.0", (27, synth.SPVCNN_IN, w[0])), ("stem.1", (27, w[0], w[0]))]

    def res(name, cin, cout):
        out.extend([(name + ".a", (27, cin, cout)), (name + ".b", (27, cout, cout))])
        if cin != cout:
            out.append((name + ".sc", (cin, cout)))

    for s in range(1, 5):
        out.append((f"down.{s}", (8, w[s - 1], w[s - 1])))
        res(f"enc.{s}.0", w[s - 1], w[s])
        res(f"enc.{s}.1", w[s], w[s])
    for u in range(1, 5):
        out.append((f"up.{u}", (8, w[3 + u], w[4 + u])))
        res(f"dec.{u}.0", w[4 + u] + w[4 - u], w[4 + u])
        res(f"dec.{u}.1", w[4 + u], w[4 + u])
    for i, (cin, cout) in enumerate([(synth.SPVCNN_IN, w[0]), (w[0], w[4]), (w[4], w[6]), (w[6], w[8])]):
        out.append((f"point.{i}", (cin, cout)))
    return out + [("head", (w[8], synth.SPVCNN_CLASSES))]


def data(case, seed):
    """Points, features and weights of a case as tensors: what prepare() hands over and exact() computes on."""
    xyz, batch = cloud(case, seed)
    n, path = len(xyz), case["path"]
    d = dict(xyz=torch.from_numpy(xyz).cuda(), batch=None if batch is None else torch.from_numpy(batch).cuda())
    r = Draws(seed)
    dt = DTYPES[case.get("dtype", "bf16")]
    if path == "block":
        C = case["channels"]
        d.update(feat=r.normal(n, C, dtype=dt), convs=[(r.weight(27, C, C, dtype=dt), *r.bn(C)) for _ in range(2)],
                 Wp=r.weight(C, C, dtype=dt), bn=r.bn(C))
    elif path == "net":
        intensity = torch.rand(n, 1, generator=r.gen, device="cuda")
        d.update(feat=torch.cat([d["xyz"], intensity], 1).to(dt), P={})
        for name, shape in layers():
            sc, sh = r.bn(shape[-1])
            d["P"][name] = (r.weight(*shape, dtype=dt), None if name == "head" else sc, sh)
    return d, r, dt


def layer_data(case, d, r, dt, n, m, mc):
    """Adds the features, weights and gradients of a layer on m voxels (mc at the next stride) to d."""
    path = case["path"]
    if path == "conv":
        d.update(W=r.weight(27, case["cin"], case["cout"], dtype=dt), bn=r.bn(case["cout"]),
                 x=r.normal(m, case["cin"], dtype=dt),
                 res=r.normal(m, case["cout"], dtype=dt) if case["residual"] else None)
    elif path == "updown":
        f, c = case["fine"], case["coarse"]
        d.update(W=r.weight(8, f, c, dtype=dt), Wt=r.weight(8, c, f, dtype=dt), bn=r.bn(c), bn_t=r.bn(f),
                 x=r.normal(m, f, dtype=dt), m=m, mc=mc)
    elif path == "train_conv":
        cin, cout = case["cin"], case["cout"]
        d.update(W=r.weight(27, cin, cout, dtype=dt), bn=r.bn(cout), x=r.normal(m, cin, dtype=dt),
                 dy=r.normal(m, cout, dtype=dt), a=r.normal(m, cout, dtype=dt), m=m)
    else:  # train_point
        C = case["channels"]
        d.update(z=r.normal(n, C, dtype=dt), W=r.weight(C, C, dtype=dt), bn=r.bn(C), dout=r.normal(n, C, dtype=dt),
                 dv=r.normal(m, C, dtype=dt), a=r.normal(n, C, dtype=dt), m=m)


def strides(ws, xyz, batch, voxel, top):
    """The voxel sets of strides 1 .. 2^top and the stride-2 maps between them."""
    vox = spv.spv_voxelize(ws, xyz, voxel, batch=batch)
    coords, downs = [vox.coords[: vox.m]], []
    for _ in range(top):
        km = spv.spv_kernel_map(ws, coords[-1], K=2, stride=2)
        downs.append(km)
        coords.append(km.out_coords[: int(km.m_out_dev.item())])
    return vox, coords, downs


def prepare(case, seed):
    d, r, dt = data(case, seed)
    d.update(case=case)
    path, xyz, n = case["path"], d["xyz"], d["xyz"].shape[0]
    if path == "block":
        C = case["channels"]
        d["params"] = spv.make_block_params(C, dt, case["voxel"], [(*c, True) for c in d["convs"]], d["Wp"], *d["bn"],
                                            relu_p=True, residual=case["residual"])
        d["ws"] = spv.Workspace.for_block(n, C)
        d["out"] = torch.empty(n, C, dtype=dt, device="cuda")
        return d
    if path == "net":
        from paper_2007_16100_amd.spvcnn import SPVCNN
        host = {k: tuple(None if t is None else t.view(torch.int16).cpu().numpy().view(np.uint16)
                         if t.dtype == torch.bfloat16 else t.cpu().numpy() for t in v) for k, v in d["P"].items()}
        d["net"] = SPVCNN(host, "bf16", case["voxel"])
        return d
    ws = d["ws"] = spv.Workspace.for_ops(n, 256)
    if path == "maps":
        return d
    s = case["stride"]
    _, coords, downs = strides(ws, xyz, d["batch"], 0.05, s + 1 if path == "updown" else s)
    m, mc = coords[s].shape[0], coords[-1].shape[0]
    layer_data(case, d, r, dt, n, m, mc)
    if path == "conv":
        d.update(packed=spv.spv_pack_weights(d["W"]), nbr=spv.spv_kernel_map_nbr(ws, coords[s]),
                 out=torch.empty(m, case["cout"], dtype=dt, device="cuda"))
    elif path == "updown":
        d.update(packed=spv.spv_pack_weights(d["Wt"]), map=downs[s],
                 children=spv.spv_map_children(ws, downs[s].off, downs[s].pairs, m, mc))
    elif path == "train_conv":
        km = spv.spv_kernel_map(ws, coords[s])
        d.update(nbr=spv.spv_kernel_map_nbr(ws, coords[s]), off=km.off, pairs=km.pairs[: km.total].contiguous(),
                 ws_w=spv.Workspace.for_wgrad(27, case["cin"], case["cout"]),
                 ws_e=spv.Workspace.for_epilogue_backward(m, case["cout"]))
    else:  # train_point
        C = case["channels"]
        d.update(coords=coords[s], voxel=float(np.float32(0.05) * np.float32(2 ** s)),
                 ws_d=spv.Workspace.for_devox_backward(n, m), ws_e=spv.Workspace.for_epilogue_backward(n, C),
                 ws_l=spv.Workspace.for_linear_backward(C, C))
    return d


# -- one pass ----------------------------------------------------------------

def run(state):
    return RUN[state["case"]["path"]](state)


def run_block(d):
    return spv.spv_block(d["ws"], d["params"], d["xyz"], d["feat"], batch=d["batch"], out=d["out"])


def run_net(d):
    return d["net"].forward(d["xyz"], d["feat"], d["batch"])


def run_maps(d):
    ws = d["ws"]
    vox, coords, downs = strides(ws, d["xyz"], d["batch"], d["case"]["voxel"], 4)
    out = dict(coords=coords, counts=vox.counts[: vox.m], pt2vox=vox.pt2vox,
               nbr=[spv.spv_kernel_map_nbr(ws, c) for c in coords], off=[km.off for km in downs],
               down=[km.pairs[: km.total] for km in downs],
               children=[spv.spv_map_children(ws, km.off, km.pairs, coords[s].shape[0], coords[s + 1].shape[0])
                         for s, km in enumerate(downs)])
    if d["case"]["pairs"]:
        km = spv.spv_kernel_map(ws, coords[0])
        out.update(subm_off=km.off, subm=km.pairs[: km.total])
    return out


def run_conv(d):
    return spv.spv_sparse_conv_nbr_packed(d["ws"], d["x"], d["nbr"], d["packed"], d["case"]["cout"], d["x"].shape[0],
                                          scale=d["bn"][0], shift=d["bn"][1], relu=True, res=d["res"], out=d["out"])


def run_updown(d):
    ws, km = d["ws"], d["map"]
    y = spv.spv_sparse_conv(ws, d["x"], km.off, km.pairs, d["W"], d["mc"], scale=d["bn"][0], shift=d["bn"][1],
                            relu=True)
    z = spv.spv_sparse_conv_up_packed(ws, y, d["children"], d["packed"], d["case"]["fine"], d["m"],
                                      scale=d["bn_t"][0], shift=d["bn_t"][1], relu=True)
    return dict(down=y, up=z)


def run_train_conv(d):
    ws, m, cout = d["ws"], d["m"], d["case"]["cout"]
    (sc, sh), x, W, nbr = d["bn"], d["x"], d["W"], d["nbr"]
    y = spv.spv_sparse_conv_nbr(ws, x, nbr, W, cout, m, scale=sc, shift=sh, relu=True)
    da, _, dsc, dsh = spv.spv_epilogue_backward(d["ws_e"], d["dy"], d["a"], sc, sh, True)
    dx = spv.spv_sparse_conv_dgrad_nbr(ws, da, nbr, W)
    dW = spv.spv_sparse_conv_wgrad(d["ws_w"], x, da, d["off"], d["pairs"], 27)
    return dict(y=y, da=da, dscale=dsc, dshift=dsh, dx=dx, dW=dW)


def run_train_point(d):
    ws, s, z, W, (sc, sh) = d["ws"], d["case"]["stride"], d["z"], d["W"], d["bn"]
    vox = spv.spv_voxelize_onto(ws, d["coords"], d["xyz"], d["voxel"], z, d["batch"])
    t, ci, cw = spv.spv_devoxelize(ws, d["coords"], vox.vfeat, d["xyz"], 0.05, s, batch=d["batch"], want_corners=True)
    out = spv.spv_linear(ws, z, W, scale=sc, shift=sh, relu=True, res=t, res_after_act=True)
    da, dt, dsc, dsh = spv.spv_epilogue_backward(d["ws_e"], d["dout"], d["a"], sc, sh, True, res=t, res_after_act=True)
    dz, dW = spv.spv_linear_backward(d["ws_l"], z, W, da)
    dvfeat = spv.spv_devoxelize_backward(d["ws_d"], ci, cw, dt, d["m"])
    dfeat = spv.spv_voxelize_backward(d["dv"], vox.counts, vox.pt2vox, d["m"])
    return dict(vfeat=vox.vfeat, counts=vox.counts, out=out, dz=dz, dW=dW, dscale=dsc, dshift=dsh, dvfeat=dvfeat,
                dfeat=dfeat)


RUN = dict(block=run_block, net=run_net, maps=run_maps, conv=run_conv, updown=run_updown, train_conv=run_train_conv,
           train_point=run_train_point)


# -- what a pass cannot do without -------------------------------------------

def work(case):
    """Compulsory bytes (inputs read once, outputs written once) and operations, on the typical
    number of voxels and pairs of such a cloud."""
    n, path = case["points"], case["path"]
    b = 4 if case.get("dtype") == "f32" else 2
    coarse = case.get("voxel", 0.05) / 0.05
    m = [v * n / (1.0 if s else coarse ** 0.6) for s, v in enumerate(VOXELS)]
    if path == "block":
        C = case["channels"]
        return dict(bytes=12 * n + 2 * b * C * n + b * 55 * C * C, flops=2.0 * C * C * (2 * PAIRS[0] * m[0] + n))
    if path == "net":
        w, ops, size = synth.SPVCNN_WIDTHS, 0.0, 0
        for name, shape in layers():
            part = name.split(".")
            size += math.prod(shape)
            s = int(part[1]) if part[0] in ("enc", "down") else 4 - int(part[1]) if part[0] in ("dec", "up") else 0
            rows = {"stem": PAIRS[0] * m[0], "point": n, "head": n, "down": m[s - 1], "up": m[s]}.get(
                part[0], m[s] * (1.0 if part[-1] == "sc" else PAIRS[s]))
            ops += 2.0 * rows * shape[-2] * shape[-1]
        return dict(bytes=12 * n + 8 * n + 2 * synth.SPVCNN_CLASSES * n + 2 * size, flops=ops)
    if path == "maps":
        size = 12 * n + 4 * n + 4 * m[0] + sum(16 * v + 108 * v for v in m) + sum(
            8 * m[s] + 32 * m[s + 1] for s in range(4))
        return dict(bytes=size + (8 * PAIRS[0] * m[0] if case["pairs"] else 0), flops=0.0)
    ms, p = m[case["stride"]], PAIRS[case["stride"]] * m[case["stride"]]
    if path == "conv":
        i, o = case["cin"], case["cout"]
        return dict(bytes=b * ms * (i + o * (2 if case["residual"] else 1)) + 108 * ms + 27 * i * o * b,
                    flops=2.0 * i * o * p)
    if path == "updown":
        f, c, mc = case["fine"], case["coarse"], m[case["stride"] + 1]
        return dict(bytes=b * (2 * f * ms + 2 * c * mc) + 8 * ms + 32 * mc + 16 * f * c * b, flops=4.0 * f * c * ms)
    if path == "train_conv":
        i, o = case["cin"], case["cout"]
        return dict(bytes=b * ms * (2 * i + 4 * o) + 108 * ms + 8 * p + 27 * i * o * (b + 4), flops=3 * 2.0 * i * o * p)
    C = case["channels"]
    return dict(bytes=12 * n + b * C * (6 * n + 2 * ms) + 4 * C * ms + C * C * (b + 4), flops=3 * 2.0 * n * C * C)


def tolerance(case):
    if case["path"] == "maps":
        return "exact"
    # about four times the distance from exact() that was measured: 8e-8, 2.3e-4, 1.7e-3 to 2.2e-3 and,
    # through the whole network, 4e-3
    if case.get("dtype") == "f32":
        return {"rel": 1e-6, "max": 2e-5}
    if case.get("dtype") == "f16":
        return {"rel": 1e-3, "max": 0.02}
    return {"rel": 1.6e-2, "max": 0.5} if case["path"] == "net" else {"rel": 8e-3, "max": 0.1}


# -- the same in 64 bits, in plain torch ---------------------------------------

def pack_keys(c):
    c = c.long()
    return (c[:, 0] << 48) | ((c[:, 1] + 32768) << 32) | ((c[:, 2] + 32768) << 16) | (c[:, 3] + 32768)


def point_voxels(d, voxel):
    """(b, x, y, z) of every point: floor of the float32 quotient."""
    q = np.floor(d["xyz"].cpu().numpy() / np.float32(voxel)).astype(np.int64)
    q = torch.from_numpy(q).cuda()
    b = torch.zeros(len(q), dtype=torch.long, device="cuda") if d["batch"] is None else d["batch"].long()
    return torch.cat([b[:, None], q], 1)


def find(keys, wanted):
    """Row of each wanted key in the sorted keys, or -1."""
    at = torch.searchsorted(keys, wanted).clamp_(max=len(keys) - 1)
    return torch.where(keys[at] == wanted, at, torch.full_like(at, -1))


class Grid:
    """The voxels of a stride, in ascending order."""

    def __init__(self, coords):
        self.keys, first = torch.unique(pack_keys(coords), return_inverse=True)
        k = self.keys
        self.coords = torch.stack([k >> 48, ((k >> 32) & 65535) - 32768, ((k >> 16) & 65535) - 32768,
                                   (k & 65535) - 32768], 1)
        self.of, self.tables = first, None

    def down(self):
        c = self.coords.clone()
        c[:, 1:] = torch.div(c[:, 1:], 2, rounding_mode="floor")
        g = Grid(c)
        p = self.coords[:, 1:] & 1
        self.parent, self.child = g.of, 4 * p[:, 0] + 2 * p[:, 1] + p[:, 2]
        return g

    def pairs(self):
        if self.tables is None:
            self.tables = []
            for k in range(27):
                i = find(self.keys, self.keys + ((k // 9 - 1) << 32) + ((k // 3 % 3 - 1) << 16) + (k % 3 - 1))
                j = torch.nonzero(i >= 0)[:, 0]
                self.tables.append((i[j], j))
        return self.tables

    def conv(self, x, W):
        y = torch.zeros(len(self.keys), W.shape[2], dtype=torch.float64, device="cuda")
        for k, (i, j) in enumerate(self.pairs()):
            y[j] += x[i] @ W[k]
        return y

    def conv_down(self, x, W, coarse):
        y = torch.zeros(len(coarse.keys), W.shape[2], dtype=torch.float64, device="cuda")
        for k in range(8):
            i = torch.nonzero(self.child == k)[:, 0]
            y[self.parent[i]] += x[i] @ W[k]
        return y

    def conv_up(self, x, W):
        y = torch.empty(len(self.keys), W.shape[2], dtype=torch.float64, device="cuda")
        for k in range(8):
            i = torch.nonzero(self.child == k)[:, 0]
            y[i] = x[self.parent[i]] @ W[k]
        return y


def mean(f, of, m):
    s = torch.zeros(m, f.shape[1], dtype=torch.float64, device="cuda").index_add_(0, of, f)
    return s / torch.bincount(of, minlength=m).clamp_(min=1)[:, None]


def corners(d, grid, stride, voxel):
    """Rows [n][8] (-1 where absent) and renormalized weights [n][8] of the trilinear corners."""
    a = d["xyz"].cpu().numpy() / np.float32(voxel) * np.float32(2.0 ** -stride) - np.float32(0.5)
    base = np.floor(a)
    t = torch.from_numpy((a - base).astype(np.float64)).cuda()
    base = torch.from_numpy(base.astype(np.int64)).cuda()
    b = torch.zeros(len(base), dtype=torch.long, device="cuda") if d["batch"] is None else d["batch"].long()
    idx, w = [], []
    for c in range(8):
        o = torch.tensor([c >> 2, c >> 1 & 1, c & 1], device="cuda")
        idx.append(find(grid.keys, pack_keys(torch.cat([b[:, None], base + o], 1))))
        w.append(torch.where(o.bool(), t, 1 - t).prod(1))
    idx, w = torch.stack(idx, 1), torch.stack(w, 1)
    w = torch.where(idx >= 0, w, torch.zeros_like(w))
    s = w.sum(1, keepdim=True)
    return idx, torch.where(s > 0, w / s, torch.zeros_like(w))


def blend(vfeat, idx, w):
    return sum(vfeat[idx[:, c].clamp(min=0)] * w[:, c: c + 1] for c in range(8))


def exact(case, seed):
    if case["path"] == "maps":
        return None
    with torch.no_grad():
        return EXACT[case["path"]](case, seed)


def wide(t):
    if isinstance(t, (tuple, list)):
        return [wide(x) for x in t]
    return t.double() if isinstance(t, torch.Tensor) and t.is_floating_point() else t


def exact_block(case, seed):
    d, _, _ = data(case, seed)
    grid, feat, (sc, sh) = Grid(point_voxels(d, case["voxel"])), d["feat"].double(), wide(d["bn"])
    x = y = mean(feat, grid.of, len(grid.keys))
    for l, (W, s, h) in enumerate(wide(d["convs"])):
        y = grid.conv(y, W) * s + h + (x if case["residual"] and l == 1 else 0)
        y = y.relu()
    return blend(y, *corners(d, grid, 0, case["voxel"])) + ((feat @ d["Wp"].double()) * sc + sh).relu()


def exact_net(case, seed):
    d, _, _ = data(case, seed)
    P, feat, v = {k: wide(t) for k, t in d["P"].items()}, d["feat"].double(), case["voxel"]
    grids = [Grid(point_voxels(d, v))]
    for _ in range(4):
        grids.append(grids[-1].down())
    of = [grids[0].of]
    for g in grids[:4]:
        of.append(g.parent[of[-1]])

    def bn(y, name):
        return y * P[name][1] + P[name][2]

    def res(x, name, s):
        h = bn(grids[s].conv(x, P[name + ".a"][0]), name + ".a").relu()
        short = bn(x @ P[name + ".sc"][0], name + ".sc") if name + ".sc" in P else x
        return (bn(grids[s].conv(h, P[name + ".b"][0]), name + ".b") + short).relu()

    def fuse(x, s, z, name):
        return blend(x, *corners(d, grids[s], s, v)) + bn(z @ P[name][0], name).relu()

    def again(z, s):
        return mean(z, of[s], len(grids[s].keys))

    x = again(feat, 0)
    for name in ("stem.0", "stem.1"):
        x = bn(grids[0].conv(x, P[name][0]), name).relu()
    skips, z = [x], fuse(x, 0, feat, "point.0")
    x = again(z, 0)
    for s in range(1, 5):
        x = bn(grids[s - 1].conv_down(x, P[f"down.{s}"][0], grids[s]), f"down.{s}").relu()
        x = res(res(x, f"enc.{s}.0", s), f"enc.{s}.1", s)
        skips.append(x)
    z = fuse(x, 4, z, "point.1")

    def up(y, u):
        t = bn(grids[4 - u].conv_up(y, P[f"up.{u}"][0]), f"up.{u}").relu()
        return res(res(torch.cat([t, skips[4 - u]], 1), f"dec.{u}.0", 4 - u), f"dec.{u}.1", 4 - u)

    z = fuse(up(up(again(z, 4), 1), 2), 2, z, "point.2")
    z = fuse(up(up(again(z, 2), 3), 4), 0, z, "point.3")
    return z @ P["head"][0] + P["head"][2]


def layer_state(case, seed):
    """The tensors prepare() hands over and the voxel sets of every stride up to the next."""
    d, r, dt = data(case, seed)
    grids = [Grid(point_voxels(d, 0.05))]
    for _ in range(case["stride"] + 1):
        grids.append(grids[-1].down())
    m, mc = (len(g.keys) for g in grids[case["stride"]:])
    layer_data(case, d, r, dt, d["xyz"].shape[0], m, mc)
    return d, grids


def exact_conv(case, seed):
    d, grids = layer_state(case, seed)
    y = grids[case["stride"]].conv(d["x"].double(), d["W"].double()) * d["bn"][0] + d["bn"][1]
    return (y if d["res"] is None else y + d["res"]).relu()


def exact_updown(case, seed):
    d, grids = layer_state(case, seed)
    fine, coarse = grids[case["stride"]: case["stride"] + 2]
    y = (fine.conv_down(d["x"].double(), d["W"].double(), coarse) * d["bn"][0] + d["bn"][1]).relu()
    return dict(down=y, up=(fine.conv_up(y, d["Wt"].double()) * d["bn_t"][0] + d["bn_t"][1]).relu())


def exact_train_conv(case, seed):
    d, grids = layer_state(case, seed)
    grid, x, W, (sc, sh) = grids[case["stride"]], d["x"].double(), d["W"].double(), wide(d["bn"])
    y = (grid.conv(x, W) * sc + sh).relu()
    a = d["a"].double()
    gz = d["dy"].double() * (a * sc + sh > 0)
    da = gz * sc
    dx, dW = torch.zeros_like(x), torch.zeros_like(W)
    for k, (i, j) in enumerate(grid.pairs()):
        dx[i] += da[j] @ W[k].T
        dW[k] = x[i].T @ da[j]
    return dict(y=y, da=da, dscale=(gz * a).sum(0), dshift=gz.sum(0), dx=dx, dW=dW)


def exact_train_point(case, seed):
    d, grids = layer_state(case, seed)
    s, z, W, (sc, sh), m = case["stride"], d["z"].double(), d["W"].double(), wide(d["bn"]), d["m"]
    of = grids[0].of
    for g in grids[:s]:
        of = g.parent[of]
    vfeat = mean(z, of, m)
    idx, w = corners(d, grids[s], s, 0.05)
    a, dout = d["a"].double(), d["dout"].double()
    gz = dout * (a * sc + sh > 0)
    da = gz * sc
    dvfeat = torch.zeros(m, z.shape[1], dtype=torch.float64, device="cuda")
    for c in range(8):
        dvfeat.index_add_(0, idx[:, c].clamp(min=0), dout * w[:, c: c + 1])
    counts = torch.bincount(of, minlength=m)
    return dict(vfeat=vfeat, counts=None, out=((z @ W) * sc + sh).relu() + blend(vfeat, idx, w), dz=da @ W.T, dW=z.T @ da,
                dscale=(gz * a).sum(0), dshift=gz.sum(0), dvfeat=dvfeat,
                dfeat=d["dv"].double()[of] / counts[of][:, None])


EXACT = dict(block=exact_block, net=exact_net, conv=exact_conv, updown=exact_updown, train_conv=exact_train_conv,
             train_point=exact_train_point)
