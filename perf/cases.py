"""The calls whose speed this library is judged by.

A case is one layer of a network that trains with this library, at the sizes
of the repository's workloads or of generic layers beside them, taken through
the binding the way a training program calls it: the footprints are at hand
(the forward pass left them), the workspace and the gradients' buffers are the
program's own, and one pass is one call of

  "step"      conv_bwd_sparse, both gradients of a layer, dX masked by the
              footprint of X and blocks of an all-zero dY skipped in dW
  "dense"     conv_bwd_sparse without X's footprint (a layer after a pool,
              whose data gradient the paper leaves dense)
  "weight"    conv_bwd_sparse with dX = NULL (a network's first layer)
  "separate"  conv_bwd_data_masked, then conv_bwd_weight_sparse
  "forward"   conv_fwd_relu_mask, the producer of the footprints

Densities are shares of live (non-zero) elements.  Footprints are drawn
element by element ("iid") or as one spatially clustered field per image that
all channels share ("shared", where whole pixels die and work is skipped).
"""
import math

import torch

import paper_2109_07710_amd as cb


def _case(call, N, C, H, W, K, R, S=None, stride=1, pad=None, dtype="bf16", layout="nhwc", filters="krsc",
          x_density=0.4, dy_density=0.4, footprint="iid", name=None):
    c = dict(call=call, N=N, C=C, H=H, W=W, K=K, R=R, S=R if S is None else S, stride=stride,
             pad=R // 2 if pad is None else pad, dtype=dtype, layout=layout, filters=filters,
             x_density=x_density, dy_density=dy_density, footprint=footprint)
    return dict(c, name=name) if name else c


def listed():
    return [
        # the smallest layer of the workloads, float32: a call that is all launches and latency
        _case("step", 2, 16, 16, 16, 16, 3, dtype="f32", x_density=0.5, dy_density=0.5, name="step_f32_c16_16"),
        # the benchmark's layer (VGG conv3_2): both gradients, bound by the matrix cores
        _case("step", 32, 256, 56, 56, 256, 3, name="step_c256_56"),
        # VGG conv1_2: few channels and the largest tensors
        _case("step", 32, 64, 224, 224, 64, 3, x_density=0.5, dy_density=0.3, name="step_c64_224"),
        # VGG conv5_2: many channels and few pixels, the chip is hard to fill
        _case("step", 32, 512, 14, 14, 512, 3, x_density=0.2, dy_density=0.2, name="step_c512_14"),
        # ResNet-50 bottleneck, the pointwise layer: bound by memory
        _case("step", 64, 256, 56, 56, 64, 1, x_density=0.6, dy_density=0.45, name="step_1x1_c256to64_56"),
        # ResNet-50 bottleneck, the spatial layer
        _case("step", 64, 64, 56, 56, 64, 3, x_density=0.45, dy_density=0.3, name="step_3x3_c64_56"),
        # a downsampling layer: stride 2, the width doubled
        _case("step", 32, 128, 56, 56, 256, 3, stride=2, x_density=0.5, dy_density=0.4, name="step_stride2_c128_56"),
        # odd sizes: channels that are no power of two, an odd image, filters stored KCRS, a small batch
        _case("step", 6, 104, 35, 27, 200, 3, filters="kcrs", x_density=0.5, dy_density=0.5, name="step_ragged_c104_35x27"),
        # a caller that keeps the layouts of torch: NCHW activations, KCRS filters
        _case("step", 32, 256, 56, 56, 256, 3, layout="nchw", filters="kcrs", name="step_nchw_c256_56"),
        # float32 training of an ordinary layer
        _case("step", 16, 128, 28, 28, 128, 3, dtype="f32", x_density=0.5, dy_density=0.4, name="step_f32_c128_28"),
        # the forward pass that leaves the footprint to the backward pass
        _case("forward", 32, 256, 56, 56, 256, 3, name="forward_c256_56"),
        # the sparse end of the density sweep: whole pixels are dead, work is skipped
        _case("step", 128, 512, 14, 14, 512, 3, x_density=0.1, dy_density=0.1, footprint="shared",
              name="step_shared_c512_14"),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    while True:
        dtype = "f32" if rng.random() < 0.2 else "bf16"
        call = rng.choice(("step", "step", "step", "step", "dense", "weight", "separate", "forward"))
        R = rng.choice((1, 1, 3, 3, 3, 3, 3, 5))
        stride = 1 if call == "forward" or rng.random() < 0.75 else 2
        plain = call != "forward" and rng.random() < 0.2
        if rng.random() < 0.5:
            C, K = (rng.choice((64, 128, 256, 512)) for _ in range(2))
        else:
            C, K = (8 * _log(rng, 1, 64) for _ in range(2))
        if call == "weight":
            C = 8
        H = _log(rng, 7, 224)
        W = H if rng.random() < 0.6 else min(224, max(7, H + rng.randint(-5, 5)))
        P, Q = (H - 1) // stride + 1, (W - 1) // stride + 1
        most = {"bf16": 60e9, "f32": 2e9}[dtype] / stride ** 2 / (4 if R == 5 or C % 64 or K % 64 else 1)
        image = 2.0 * C * K * R * R * P * Q
        # the batch from one image to what the budget of one pass or 64 million elements allow
        top = min(128, int(most / image), int(64e6 / (max(C * H * W, K * P * Q))))
        if top < 1:
            continue
        case = _case(call, _log(rng, 1, top), C, H, W, K, R, stride=stride, dtype=dtype,
                     layout="nchw" if plain else "nhwc", filters="kcrs" if plain or rng.random() < 0.2 else "krsc",
                     x_density=round(rng.uniform(0.15, 0.7), 2), dy_density=round(rng.uniform(0.15, 0.7), 2),
                     footprint="shared" if rng.random() < 0.15 else "iid")
        return case


def _desc(case):
    return cb.ConvDesc.make(case["N"], case["C"], case["H"], case["W"], case["K"], case["R"], case["S"], case["stride"],
                            (case["pad"], case["pad"]), dtype=case["dtype"], w_layout=case["filters"],
                            act_layout=case["layout"])


def _field(g, kind, n, h, w, c, density):
    """A footprint [n, h, w, c] with about `density` of its elements live."""
    if kind == "iid":
        return torch.rand((n, h, w, c), generator=g, device="cuda") < density
    f = torch.randn((n, h, w), generator=g, device="cuda")
    f = sum(torch.roll(f, (i, j), (1, 2)) for i in range(-2, 3) for j in range(-2, 3))
    cut = f.flatten().sort().values[min(f.numel() - 1, int((1.0 - density) * f.numel()))]
    return (f > cut).unsqueeze(3).expand(n, h, w, c)


def _tensors(case, seed):
    """X (a ReLU output), W (He-initialised) and dY as NHWC and KRSC."""
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    N, C, H, W, K, R, S = (case[k] for k in "NCHWKRS")
    d = _desc(case)
    dt = {"bf16": torch.bfloat16, "f32": torch.float32}[case["dtype"]]
    x = torch.randn((N, H, W, C), generator=g, device="cuda").abs_()
    x.mul_(_field(g, case["footprint"], N, H, W, C, case["x_density"]))
    w = torch.randn((K, R, S, C), generator=g, device="cuda").mul_(math.sqrt(2.0 / (C * R * S)))
    dy = None
    if case["call"] != "forward":
        dy = torch.randn((N, d.P, d.Q, K), generator=g, device="cuda")
        dy = torch.where(_field(g, case["footprint"], N, d.P, d.Q, K, case["dy_density"]), dy, torch.zeros_like(dy)).to(dt)
    return x.to(dt), w.to(dt), dy


def _stored(case, x, w, dy):
    """The tensors in the layouts that the case's caller keeps."""
    if case["layout"] == "nchw":
        x, dy = (t if t is None else t.permute(0, 3, 1, 2).contiguous() for t in (x, dy))
    if case["filters"] == "kcrs":
        w = w.permute(0, 3, 1, 2).contiguous()
    return x, w, dy


def prepare(case, seed):
    desc = _desc(case)
    x, w, dy = _stored(case, *_tensors(case, seed))
    s = {"call": case["call"], "desc": desc, "x": x, "w": w}
    words = lambda n: torch.empty(n, dtype=torch.int32, device="cuda")  # noqa: E731
    if case["call"] == "forward":
        s["y"] = torch.empty((case["N"], desc.P, desc.Q, case["K"]), dtype=x.dtype, device="cuda")
        s["y_mask"] = words(cb.cbw_dy_mask_words(desc))
        s["ws"] = cb.workspace(desc, cb.CBW_OP_FWD)
        return s
    s["dy"], s["dy_mask"] = dy, words(cb.cbw_dy_mask_words(desc))
    cb.cbw_nonzero_mask_pack(desc.dtype, dy.numel(), dy, s["dy_mask"])
    s["dw"] = torch.empty_like(w, dtype=torch.float32)
    s["x_mask"] = s["dx"] = None
    if case["call"] in ("step", "separate"):
        s["x_mask"] = words(cb.cbw_mask_words(desc))
        cb.cbw_relu_mask_pack(desc, x, s["x_mask"])
    if case["call"] != "weight":
        s["dx"] = torch.empty_like(x)
    if case["call"] == "separate":
        s["ws"] = cb.workspace(desc, cb.CBW_OP_BWD_DATA_MASKED)
        s["ws_weight"] = cb.workspace(desc, cb.CBW_OP_BWD_WEIGHT)
    else:
        s["ws"] = cb.workspace(desc, cb.CBW_OP_BWD_BOTH)
    return s


def run(s):
    if s["call"] == "forward":
        cb.conv_fwd_relu_mask(s["desc"], s["x"], s["w"], s["y"], s["y_mask"], s["ws"])
        return {"y": s["y"], "y_mask": s["y_mask"]}
    if s["call"] == "separate":
        cb.conv_bwd_data_masked(s["desc"], s["dy"], s["w"], s["x_mask"], s["dx"], s["ws"])
        cb.conv_bwd_weight_sparse(s["desc"], s["x"], s["dy"], s["dy_mask"], s["dw"], s["ws_weight"])
        return {"dx": s["dx"], "dw": s["dw"]}
    w = s["w"] if s["dx"] is not None else None
    cb.conv_bwd_sparse(s["desc"], s["x"], s["dy"], w, s["x_mask"], s["dy_mask"], s["dx"], s["dw"], s["ws"])
    return {"dw": s["dw"]} if s["dx"] is None else {"dx": s["dx"], "dw": s["dw"]}


def work(case):
    """Every tensor once; two operations a multiply-add of the dense products that land inside the image.  With element-wise
    footprints no whole row or block of the matrix products is dead; with a shared one the dead pixels' products are not
    needed: dX's where X is dead or dY is, dW's likewise."""
    d, b = _desc(case), {"bf16": 2, "f32": 4}[case["dtype"]]
    N, C, H, W, K, R, S = (case[k] for k in "NCHWKRS")
    x, y, w = N * H * W * C, N * d.P * d.Q * K, K * R * S * C

    def taps(size, out, f):
        return sum(0 <= p * case["stride"] - case["pad"] + r < size for p in range(out) for r in range(f))

    product = 2.0 * N * C * K * taps(H, d.P, R) * taps(W, d.Q, S)
    if case["call"] == "forward":
        return {"bytes": (x + w + y) * b + y / 8, "flops": product}
    if case["footprint"] == "shared":
        product *= case["dy_density"] * (case["x_density"] if case["call"] != "dense" else 1.0)
    if case["call"] == "weight":
        return {"bytes": (x + y) * b + 4 * w + y / 8, "flops": product}
    mask = x / 8 if case["call"] in ("step", "separate") else 0
    return {"bytes": (2 * x + y + w) * b + 4 * w + y / 8 + mask, "flops": 2 * product}


def tolerance(case):
    """bf16: dX and Y are rounded to 8 bits of significand (relative error 2^-9 at most, 1.7e-3 in the 2-norm against 64 bits),
    and another order of the float32 sums moves a value to its neighbour, 2^-8 of it at most.  A footprint word differs where
    a sum next to zero changes its sign.  float32: the sums' own rounding, up to 2.4e-7 in the 2-norm
    against 64 bits."""
    if case["dtype"] == "f32":
        return {"rel": 1e-6, "max": 4e-5, "differ": 2e-4}
    return {"rel": 7e-3, "max": 2e-2, "differ": 2e-4}


def _taps(case, d):
    """For each filter tap: the slices of the output pixels and of the input pixels it joins."""
    st, pad = case["stride"], case["pad"]

    def axis(size, out, f):
        lo = max(0, -((f - pad) // st))                 # first output whose input is >= 0
        hi = min(out - 1, (size - 1 + pad - f) // st)   # last output whose input is < size
        first = lo * st - pad + f
        return (slice(lo, hi + 1), slice(first, first + (hi - lo) * st + 1, st)) if hi >= lo else None

    for r in range(case["R"]):
        for s in range(case["S"]):
            a, b = axis(case["H"], d.P, r), axis(case["W"], d.Q, s)
            if a and b:
                yield r, s, (slice(None), a[0], b[0]), (slice(None), a[1], b[1])


def exact(case, seed):
    d = _desc(case)
    x16, w, dy = _tensors(case, seed)
    x, w = x16.double(), w.double()
    dy = None if dy is None else dy.double()
    C, K = case["C"], case["K"]
    if case["call"] == "forward":
        y = torch.zeros((case["N"], d.P, d.Q, K), dtype=torch.float64, device="cuda")
        for r, s, out, inp in _taps(case, d):
            a = x[inp].contiguous()
            y[out] += (a.view(-1, C) @ w[:, r, s].t().contiguous()).view(*a.shape[:3], K)
        y.clamp_(min=0.0)
        bits = (y > 0).flatten()
        bits = torch.nn.functional.pad(bits, (0, -bits.numel() % 32)).view(-1, 32).to(torch.int64)
        bits = (bits << torch.arange(32, device="cuda")).sum(1)
        return {"y": y, "y_mask": torch.where(bits >= 1 << 31, bits - (1 << 32), bits).to(torch.int32)}
    dx, dw = torch.zeros_like(x), torch.zeros_like(w)
    for r, s, out, inp in _taps(case, d):
        g, a = dy[out].contiguous(), x[inp].contiguous()
        dw[:, r, s] = g.view(-1, K).t().contiguous() @ a.view(-1, C)
        if case["call"] != "weight":
            dx[inp] += (g.view(-1, K) @ w[:, r, s].contiguous()).view(a.shape)
    if case["call"] in ("step", "separate"):
        dx.mul_(x16 > 0)
    dx, dw, _ = _stored(case, dx, dw, None)
    return {"dw": dw} if case["call"] == "weight" else {"dx": dx, "dw": dw}
