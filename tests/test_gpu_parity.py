"""GPU parity: the HIP path (through the C ABI) against the CPU oracle, element by element.

Bar: routing indices, counts and active lists bit-exact; gate weights |d| <= 1e-6; layer outputs
max|d| / max|ref| <= 5e-3 for bf16 storage (fp32 accumulation; the hidden vector is rounded to bf16
as a bf16 model does) and <= 2e-5 for fp32 storage.

Routing is a function of the fp32 logits.  The library accumulates them in fp64 like the oracle, so
they are expected to agree bit for bit; should a logit ever differ (summation order, last place),
the test still requires (i) |d| within one fp32 ulp and (ii) routing identical to the oracle's
routing OF THE LOGITS THE GPU USED, and compares the output under that routing.
"""
import ctypes
import sys

import numpy as np
import pytest

from paper_2511_02237_amd import workloads as W

pytestmark = pytest.mark.gpu

TOL = {"bf16": 5e-3, "f32": 2e-5}


@pytest.fixture(scope="module")
def torch():
    import torch as _t
    assert _t.cuda.is_available(), "no GPU visible"
    return _t


@pytest.fixture(scope="module")
def B_():
    from paper_2511_02237_amd import binding
    binding.lib()  # raises if the HIP library is missing
    return binding


def say(*a):
    print(*a, flush=True)
    sys.stdout.flush()


def route_gpu(torch, B_, lg, k, k0):
    res = B_.oea_route(torch.from_numpy(lg).cuda(), k, k0)
    torch.cuda.synchronize()
    return {n: v.cpu().numpy() for n, v in res.items()}


def assert_routing_equal(got, ref, ctx):
    assert int(got["n_active"][0] if np.ndim(got["n_active"]) else got["n_active"]) == ref["n_active"], ctx
    assert np.array_equal(got["active_list"], ref["active_list"]), ctx
    assert np.array_equal(got["n_sel"], ref["n_sel"]), ctx
    assert np.array_equal(got["expert_idx"], ref["expert_idx"]), ctx
    assert np.abs(got["gate_w"].astype(np.float64) - ref["gate_w"]).max() <= 1e-6, ctx


ROUTE_CASES = [(B, N, k, k0, kind, seed)
               for (B, N, k) in [(4, 16, 4), (16, 128, 8), (3, 7, 5), (33, 64, 6), (1, 128, 8), (128, 128, 8),
                                 (16, 100, 8), (7, 200, 12), (5, 512, 32), (200, 130, 8), (16, 1, 1),
                                 # several token groups with the keys kept in registers between the phases
                                 (70, 64, 6), (100, 128, 8), (127, 128, 8), (256, 128, 8),
                                 (1024, 128, 8), (1024, 512, 32)]  # the last two: the size limits of the entry point
               for k0 in sorted({1, max(1, k // 2), k})
               for kind in W.LOGIT_KINDS
               for seed in (0, 1)]


def test_route_bit_exact(torch, B_, oracle):
    n = 0
    for (B, N, k, k0, kind, seed) in ROUTE_CASES:
        ctx = "route B=%d N=%d k=%d k0=%d kind=%s seed=%d" % (B, N, k, k0, kind, seed)
        lg = W.make_logits(B, N, seed, kind)
        got = route_gpu(torch, B_, lg, k, k0)
        assert_routing_equal(got, oracle.route(lg, k, k0), ctx)
        n += 1
    say("route cases checked:", n)


def test_route_many_seeds_qwen_shape(torch, B_, oracle):
    for seed in range(64):
        lg = W.make_logits(16, 128, 9000 + seed, "gaussian" if seed % 2 == 0 else "skew")
        for k0 in (1, 3, 5, 8):
            assert_routing_equal(route_gpu(torch, B_, lg, 8, k0), oracle.route(lg, 8, k0), "seed %d k0 %d" % (seed, k0))


def test_route_non_finite_logits_stay_in_range(torch, B_):
    lg = W.make_logits(16, 128, 5, "gaussian")
    lg[0, :5] = np.nan
    lg[1, 3] = np.inf
    lg[2, :] = -np.inf
    lg[3, :] = np.nan
    got = route_gpu(torch, B_, lg, 8, 3)
    idx = got["expert_idx"]
    assert ((idx >= -1) & (idx < 128)).all()
    T = int(got["n_active"][0])
    assert 0 < T <= 128 and ((got["active_list"][:T] >= 0) & (got["active_list"][:T] < 128)).all()
    assert (got["n_sel"] >= 0).all() and (got["n_sel"] <= 8).all()


def run_layer(torch, B_, L, k0, ws=None, bias=None, mask=None, path=None):
    dev = {f: B_.to_device(getattr(L, f)) for f in ("x", "w_router", "w_gate", "w_up", "w_down")}
    return run_layer_dev(torch, B_, L, dev, k0, ws, bias, mask, path)


def run_layer_dev(torch, B_, L, dev, k0, ws=None, bias=None, mask=None, path=None):
    """path: kernel path of oea_test_opts (None = the product entry point, automatic choice)."""
    if ws is None:
        ws = B_.new_workspace(L.B, L.d, L.N, L.I, L.k)
    out, tap = B_.moe_decode(dev["x"], dev["w_router"], dev["w_gate"], dev["w_up"], dev["w_down"], L.k, k0, ws,
                             router_bias=None if bias is None else torch.from_numpy(bias).cuda(),
                             token_mask=None if mask is None else torch.from_numpy(mask).cuda(), taps=True,
                             kernel_path=path)
    torch.cuda.synchronize()
    return out.cpu().numpy(), {n: v.cpu().numpy() for n, v in tap.items()}


def check_layer(oracle, L, k0, out, tap, ctx, bias=None, mask=None):
    ref = oracle.moe_decode(L.x, L.w_router, L.w_gate, L.w_up, L.w_down, L.k, k0, router_bias=bias,
                            token_mask=mask)
    lg_gpu, lg_ref = tap["logits"], ref["logits"]
    same_bits = np.array_equal(lg_gpu.view(np.uint32), lg_ref.view(np.uint32))
    if not same_bits:
        ulp = np.spacing(np.abs(lg_ref))
        assert (np.abs(lg_gpu.astype(np.float64) - lg_ref.astype(np.float64)) <= ulp).all(), ctx
        say("note: %s: %d logits differ in the last place" % (ctx, int((lg_gpu != lg_ref).sum())))
    # routing is exact as a function of the logits the GPU used
    r_gpu_logits = oracle.route(lg_gpu, L.k, k0, token_mask=mask)
    assert_routing_equal(tap, r_gpu_logits, ctx)
    if same_bits or np.array_equal(r_gpu_logits["expert_idx"], ref["expert_idx"]):
        ref_out = ref["out"]
    else:  # a last-place logit difference flipped a near-tie: compare under the GPU's routing
        ref_out = oracle.moe_combine(L.x, L.w_gate, L.w_up, L.w_down, r_gpu_logits["expert_idx"],
                                     r_gpu_logits["gate_w"])
    scale = np.abs(ref_out).max()
    err = np.abs(out.astype(np.float64) - ref_out).max() / scale
    assert np.isfinite(out).all(), ctx
    assert err <= TOL[L.dtype], "%s: max|d|/max|ref| = %.3e" % (ctx, err)
    return err, ref


@pytest.mark.parametrize("name", ["toy", "mid_bf16", "mid_f32"])
def test_small_layers_all_k0(torch, B_, oracle, name):
    for seed in range(32):
        L = W.make_layer(name, 100 + seed)
        for k0 in L.k0s:
            ctx = "%s seed=%d k0=%d" % (name, seed, k0)
            out, tap = run_layer(torch, B_, L, k0)
            err, _ = check_layer(oracle, L, k0, out, tap, ctx)
            if seed < 2:
                say(ctx, "T=%d err=%.2e" % (int(tap["n_active"][0]), err))


@pytest.mark.parametrize("B", [1, 2, 5, 16, 33, 64, 300, 1024])  # 1024: the batch limit of the entry point
def test_batch_sizes_mid_shape(torch, B_, oracle, B):
    L = W.make_layer("mid_bf16", 200 + B, B=B)
    for k0 in (1, 3, 6):
        out, tap = run_layer(torch, B_, L, k0)
        check_layer(oracle, L, k0, out, tap, "mid_bf16 B=%d k0=%d" % (B, k0))


def test_ragged_shapes(torch, B_, oracle):
    # d, I multiples of 8 only: ragged last chunk in both stages; N not a multiple of 32 or 64
    for (d, I, N, B, k, dtype) in [(8, 8, 3, 2, 2, "bf16"), (72, 24, 5, 3, 3, "bf16"), (136, 264, 9, 6, 4, "bf16"),
                                   (24, 40, 7, 4, 3, "f32"), (1032, 520, 6, 3, 2, "bf16"), (2056, 8, 4, 2, 2, "bf16"),
                                   (520, 1032, 6, 3, 2, "f32"),
                                   # more tokens per expert than fit in LDS at once: several passes
                                   (2048, 64, 4, 80, 2, "bf16"), (4096, 16, 2, 40, 2, "bf16"),
                                   # exact 6- and 8-chunk rows at every lanes-per-row, more pairs than the unrolled 8
                                   (768, 1024, 3, 12, 3, "bf16"), (1536, 2048, 3, 12, 3, "bf16"),
                                   (3072, 4096, 2, 9, 2, "bf16"), (4096, 3072, 2, 3, 2, "bf16"),
                                   (5000, 4104, 2, 3, 2, "bf16"), (384, 512, 3, 5, 2, "f32"), (2048, 1024, 2, 3, 2, "f32")]:
        L = W.make_layer("toy", 300, d=d, I=I, N=N, B=B, k=k, dtype=dtype)
        for k0 in (1, k):
            out, tap = run_layer(torch, B_, L, k0)
            check_layer(oracle, L, k0, out, tap, "ragged d=%d I=%d N=%d B=%d k0=%d %s" % (d, I, N, B, k0, dtype))


STAGE_SHAPES = [  # (B, d, N, I, k, k0, dtype, deterministic)
    # rows covered exactly by 8, 16, 32 and 64 lanes; one granule less and one more than such a row
    (5, 192, 9, 384, 3, 2, "bf16", False), (16, 768, 5, 192, 4, 2, "bf16", False), (3, 1536, 4, 1024, 2, 1, "bf16", False),
    (4, 4096, 3, 2048, 2, 2, "bf16", False), (6, 184, 9, 392, 3, 2, "bf16", True), (6, 200, 9, 376, 3, 2, "bf16", False),
    (9, 2040, 5, 1032, 3, 1, "bf16", False), (2, 4088, 3, 2056, 2, 1, "bf16", False), (7, 8, 6, 8, 2, 1, "bf16", False),
    (5, 96, 9, 192, 3, 2, "f32", False), (7, 104, 24, 88, 5, 2, "f32", True), (3, 2048, 4, 1024, 2, 2, "f32", False),
    (6, 520, 7, 1016, 4, 3, "f32", False),
    # all of x staged (64 KB), just too much for that, and vectors in several pieces of one expert
    (32, 1024, 40, 64, 4, 2, "bf16", False), (33, 1024, 40, 64, 4, 2, "bf16", False), (90, 2048, 2, 64, 2, 1, "bf16", False),
    # more experts than one step of the row cut, three of them in a workgroup's rows, a share that could reach a fourth
    # (other kernels then), more pairs than threads
    (64, 64, 300, 32, 6, 4, "bf16", False), (60, 72, 400, 24, 8, 8, "f32", False), (60, 64, 400, 32, 8, 8, "bf16", True),
    (40, 72, 512, 24, 8, 8, "f32", False), (300, 64, 3, 40, 2, 2, "bf16", True)]


def experts_in_a_share(expert_idx, rows, beta, n_wg):
    """Most experts that one workgroup's rows belong to when the rows (cost 64 + beta x pairs of their expert) are
    shared by cost."""
    cost = 64.0 + beta * np.unique(expert_idx[expert_idx >= 0], return_counts=True)[1]
    ends = np.concatenate([[0.0], np.cumsum(cost)])
    cut = ends[-1] * np.arange(n_wg + 1) / n_wg
    e = np.minimum(np.searchsorted(ends, cut, side="right") - 1, cost.size - 1)
    first = e * rows + ((cut - ends[e]) / cost[e] * rows).astype(int)
    last = first[1:] - 1
    return int((last // rows - first[:-1] // rows + 1)[last >= first[:-1]].max())


def expert_kernels(torch, B_, dev, k, k0, ws, path, deterministic, token_mask=None, top_p=None, max_p=None):
    """The kernels that a call's two expert stages run on (oea_test_opts.h_kernels)."""
    args, _, shape = B_._layer_args(*(dev[f] for f in ("x", "w_router", "w_gate", "w_up", "w_down")), k, k0, None)
    ex, _ = B_._extras(shape, k, "cuda", None, token_mask, False, top_p, max_p, deterministic=deterministic)
    kernels = (ctypes.c_int32 * 2)(-1, -1)
    opts = B_.test_opts(kernel_path=path, kernels=kernels)
    B_._check(B_.lib().moe_decode_test(*args, B_._ptr(ws), ws.numel(), B_._stream(None),
                                       None if ex is None else ctypes.byref(ex), ctypes.byref(opts)))
    torch.cuda.synchronize()
    return list(kernels)


@pytest.mark.parametrize("shape", STAGE_SHAPES, ids=lambda c: "B%d-d%d-N%d-I%d-k%d-k0%d-%s%s" % (c[:7] + ("-det" if c[7] else "",)))
def test_stage_kernel_shapes(torch, B_, oracle, shape):
    """The dot-product stage kernels on the row lengths where their tiles change, with the vectors staged whole, per
    pair and in pieces; a padding token in every batch.  They take a layer if no workgroup's share of the rows can
    reach a fourth expert."""
    B, d, N, I, k, k0, dtype, det = shape
    L = W.make_layer("toy", 700 + B, d=d, I=I, N=N, B=B, k=k, dtype=dtype)
    mask = np.ones(B, np.uint8)
    mask[B // 2] = 0
    ws = B_.new_workspace(B, d, N, I, k, deterministic=det)
    dev = {f: B_.to_device(getattr(L, f)) for f in ("x", "w_router", "w_gate", "w_up", "w_down")}
    n_wg = torch.cuda.get_device_properties(0).multi_processor_count
    taken = 3 if (64 * N + 12 * B * k) // (n_wg * (64 + 3)) < 2 else 1
    assert expert_kernels(torch, B_, dev, k, k0, ws, 3, det) == [taken, taken]
    outs = []
    for _ in range(2):
        out, tap = B_.moe_decode(dev["x"], dev["w_router"], dev["w_gate"], dev["w_up"], dev["w_down"], k, k0, ws, taps=True,
                                 token_mask=torch.from_numpy(mask).cuda(), deterministic=det, kernel_path=3)
        torch.cuda.synchronize()
        if N == 400:
            assert taken == 3 and experts_in_a_share(tap["expert_idx"].cpu().numpy(), d, 12, n_wg) == 3
        outs.append(out.cpu().numpy())
        check_layer(oracle, L, k0, outs[-1], {n: v.cpu().numpy() for n, v in tap.items()}, str(shape), mask=mask)
    if det:
        assert np.array_equal(outs[0].view(np.uint32), outs[1].view(np.uint32))


@pytest.mark.parametrize("shape", [
    (3, 448, 40, 720, 5, 2, "f32", [1, 1]), (11, 80, 64, 656, 3, 3, "bf16", [3, 1]), (10, 1168, 40, 48, 7, 2, "bf16", [1, 3]),
    (13, 448, 24, 160, 8, 4, "f32", [3, 3]),
    # work enough, but more pairs per expert than the stage kernels stage at once
    (42, 624, 16, 152, 7, 3, "f32", [1, 3]),
    # little work, but more vectors than the streaming kernels can stage
    (50, 4096, 8, 16, 1, 1, "bf16", [3, 3])], ids=lambda c: "B%d-d%d-N%d-I%d-k%d-k0%d-%s" % c[:7])
def test_kernels_chosen_per_stage(torch, B_, oracle, shape):
    """Each stage of a layer outside the single kernel takes the streaming or the stage kernels by its own size; all
    four pairs of them give the layer."""
    B, d, N, I, k, k0, dtype, kernels = shape
    L = W.make_layer("toy", 1100 + B, d=d, I=I, N=N, B=B, k=k, dtype=dtype)
    dev = {f: B_.to_device(getattr(L, f)) for f in ("x", "w_router", "w_gate", "w_up", "w_down")}
    assert expert_kernels(torch, B_, dev, k, k0, B_.new_workspace(B, d, N, I, k), None, False) == kernels
    out, tap = run_layer_dev(torch, B_, L, dev, k0)
    check_layer(oracle, L, k0, out, tap, str(shape))


SHARE = (4096, 128, 192, 8)  # the 235B layer's share of one of eight GPUs
D30, D235 = (2048, 128, 768, 8), (4096, 128, 1536, 8)


@pytest.mark.parametrize("layer,B,k0,opts,kernels", [
    # matrix cores where an active expert serves enough pairs, and above the single kernel's batches
    (SHARE, 64, 3, {}, "matrix"), (SHARE, 8, 3, {}, "dot"), (SHARE, 200, 3, {}, "matrix"), ((512, 60, 512, 8), 32, 3, {}, "matrix"),
    ((512, 60, 512, 8), 4, 1, {}, "dot"), (D30, 16, 3, {}, "single"), (D30, 128, 3, {}, "single"), (D30, 96, 1, {}, "matrix"),
    (D30, 129, 3, {}, "matrix"), (D235, 16, 5, {}, "single"), (D235, 96, 3, {}, "matrix"),
    # (in multiples of 256 and 128 always above them, also with about one pair to an expert)
    ((2048, 512, 384, 1), 130, 1, {}, "matrix"), ((2048, 512, 384, 1), 128, 1, {}, "dot"), ((2048, 512, 320, 1), 130, 1, {}, "dot"),
    # the single kernel's d and I with more experts, or more of them per token, than it takes
    ((2048, 160, 768, 8), 64, 3, {}, "dot"), ((2048, 160, 768, 8), 128, 3, {}, "matrix"), ((2048, 128, 768, 20), 32, 3, {}, "matrix"),
    ((4096, 128, 1536, 20), 32, 3, {}, "matrix"), ((4096, 128, 1536, 16), 64, 8, {}, "matrix"),
    # experts of all tokens' own choice, few pairs on each; large experts
    (D235, 80, 8, {}, "single"), (D235, 80, 3, {}, "matrix"), (D235, 72, 3, {}, "single"), (D235, 96, 8, {}, "matrix"), (D235, 48, 2, {}, "single"), (D235, 48, 1, {}, "matrix"),
    ((4096, 128, 1024, 8), 32, 3, {}, "dot"), ((4096, 128, 1024, 8), 64, 3, {}, "matrix"), ((5120, 64, 512, 8), 24, 3, {}, "matrix"),
    # with the deterministic combine above B = 128 alone
    (D235, 128, 3, dict(deterministic=True), "single"), (D235, 129, 3, dict(deterministic=True), "matrix"),
    (SHARE, 128, 3, dict(deterministic=True), "dot"), (SHARE, 129, 3, dict(deterministic=True), "matrix"),
    # with a padding mask the live tokens may be few: matrix cores above the single kernel's batches only
    (SHARE, 64, 3, dict(live=4), "dot"), (SHARE, 64, 3, dict(live=64), "dot"), (SHARE, 200, 3, dict(live=8), "dot"),
    (D235, 128, 3, dict(live=16), "single"), (D235, 48, 1, dict(live=4), "single"), (D235, 129, 3, dict(live=129), "matrix"),
    ((512, 60, 512, 8), 32, 3, dict(live=3), "dot"), ((4096, 128, 384, 8), 129, 3, dict(live=129), "matrix"),
    # a narrow rank window leaves few pairs to an expert, a wide one does not
    (D235, 128, 3, dict(max_p=3), "single"), (D235, 128, 3, dict(max_p=24), "matrix"), (D235, 64, 1, dict(max_p=2), "single"),
    (D30, 128, 1, dict(max_p=2), "single"), (SHARE, 100, 3, dict(max_p=3), "dot"), (SHARE, 100, 3, dict(max_p=8), "matrix"),
    ((64, 16, 64, 16), 20, 16, dict(max_p=8), "matrix"),
    # a top-p cut leaves a baseline of one to k0 experts
    (SHARE, 48, 5, dict(top_p=0.1), "matrix"), (SHARE, 14, 8, dict(top_p=0.1), "dot"), (SHARE, 48, 5, dict(top_p=0.1, max_p=6), "dot"),
    ((512, 60, 512, 8), 32, 3, dict(top_p=0.1), "matrix"),
], ids=lambda v: "-".join(map(str, v)) if isinstance(v, tuple) else "-".join("%s=%s" % i for i in v.items()) if isinstance(v, dict) else str(v))
def test_kernels_chosen_automatically(torch, B_, layer, B, k0, opts, kernels):
    """The automatic choice between the single kernel, the dot-product kernels and the matrix cores, on both sides of its
    lines, for the forms that a call can have."""
    d, N, I, k = layer
    opts = dict(opts)
    live = opts.pop("live", None)
    if live is not None:
        opts["token_mask"] = (torch.arange(B, device="cuda") < live).to(torch.uint8)
    det = opts.pop("deterministic", False)
    dev = {f: torch.zeros(s, dtype=torch.bfloat16, device="cuda")
           for f, s in (("x", (B, d)), ("w_router", (N, d)), ("w_gate", (N, I, d)), ("w_up", (N, I, d)), ("w_down", (N, d, I)))}
    ws = B_.new_workspace(B, d, N, I, k, deterministic=det)
    got = expert_kernels(torch, B_, dev, k, k0, ws, None, det, **opts)
    if kernels == "dot":
        assert set(got) <= {1, 3}, got
    else:
        assert got == {"single": [0, 0], "matrix": [4, 4]}[kernels], got


@pytest.mark.parametrize("shape", [(129, 8, 3, "bf16"), (144, 32, 16, "bf16"), (145, 264, 17, "f32"), (160, 1032, 130, "bf16"),
                                   (131, 4096, 33, "bf16"), (250, 2056, 64, "f32"), (1024, 40, 512, "bf16")],
                         ids=lambda c: "B%d-d%d-N%d-%s" % c)
def test_large_batch_router_logits(torch, B_, oracle, shape):
    """The router logits of batches above 128: tiles of 16 tokens x 16 experts with remainders in both, an inner
    dimension shorter than its eight shares, ragged against a step's 64 bytes per row, and long."""
    B, d, N, dtype = shape
    L = W.make_layer("toy", 900 + B, d=d, I=8, N=N, B=B, k=2, dtype=dtype)
    bias = np.linspace(-0.5, 0.5, N).astype(np.float32)
    out, tap = run_layer(torch, B_, L, 1, bias=bias)
    check_layer(oracle, L, 1, out, tap, str(shape), bias=bias)


@pytest.mark.parametrize("bits", [0xFFFF, 0x7FC0, 0x7F80, 0xFF80], ids=lambda b: "%04x" % b)
def test_single_kernel_hidden_units_that_are_not_numbers(torch, B_, bits):
    """The single-kernel layer waits for hidden units by their bits, one NaN pattern of which means "not written
    yet": a token of NaNs (every pattern) or infinities ends without a wait running out, at its own expense only."""
    L, dev = big_layer(B_, "qwen3_30b", 2000)
    b = 5
    x = np.ascontiguousarray(L.x[:b]).copy()
    x[3] = bits
    ws = B_.new_workspace(b, L.d, L.N, L.I, L.k)
    for _ in range(3):
        out = B_.moe_decode(B_.to_device(x), dev["w_router"], dev["w_gate"], dev["w_up"], dev["w_down"], L.k, 3, ws)
    B_.workspace_check(ws)
    out = out.cpu().numpy()
    assert np.isfinite(out[[0, 1, 2, 4]]).all() and not np.isfinite(out[3]).any()


@pytest.mark.parametrize("path,b", [(None, 5), (None, 40), (1, 5), (2, 5), (3, 5), (4, 5)],
                         ids=["single", "single-gather", "generic", "stream", "stage", "matrix"])
def test_activation_over_its_whole_range(torch, B_, path, b):
    """silu(g) u for gate sums down to -88.5, where 1 + exp(-g) leaves the range whose reciprocal is a normal number:
    every kernel divides.  Column 0 of W_gate and W_up holds the sums themselves and W_down copies
    hidden unit c to output c.  Tolerance: 2^-9 for the hidden unit's rounding to bf16, and 2^-9 above the 1e-5 that
    the fast exponential of 88 can be off."""
    d, N, I = 2048, 4, 768
    g = -0.5 * torch.arange(I, device="cuda").remainder(178).float()  # 0 ... -88.5, exact in bf16
    x = torch.zeros((b, d), dtype=torch.bfloat16, device="cuda")
    x[:, 0] = 1.0
    w_router = torch.zeros((N, d), dtype=torch.bfloat16, device="cuda")
    w_gate = torch.zeros((N, I, d), dtype=torch.bfloat16, device="cuda")
    w_gate[:, :, 0] = g.bfloat16()
    w_up = torch.zeros_like(w_gate)
    w_up[:, :, 0] = 1.0
    w_down = torch.zeros((N, d, I), dtype=torch.bfloat16, device="cuda")
    w_down[:, torch.arange(I), torch.arange(I)] = 1.0
    ws = B_.new_workspace(b, d, N, I, 1)
    dev = dict(x=x, w_router=w_router, w_gate=w_gate, w_up=w_up, w_down=w_down)
    assert expert_kernels(torch, B_, dev, 1, 1, ws, path, False) == [{None: 0, 2: 1}.get(path, path)] * 2
    out = B_.moe_decode(x, w_router, w_gate, w_up, w_down, 1, 1, ws, kernel_path=path)
    torch.cuda.synchronize()
    ref = torch.zeros(d, dtype=torch.float64, device="cuda")
    ref[:I] = g.double() / (1 + torch.exp(-g.double()))
    assert ((out.double() - ref).abs() <= 2.0 ** -8 * ref.abs()).all()


def test_generic_kernel_path(torch, B_, oracle):
    """The generic expert kernels (used when the staged token vectors do not fit in LDS) on shapes the
    automatic choice would give to the streaming kernels."""
    for name, seed in (("toy", 600), ("mid_bf16", 601), ("mid_f32", 602)):
        L = W.make_layer(name, seed)
        for k0 in L.k0s:
            out, tap = run_layer(torch, B_, L, k0, path=1)
            check_layer(oracle, L, k0, out, tap, "generic %s k0=%d" % (name, k0))
    for (d, I, N, B, k, dtype) in [(72, 24, 5, 3, 3, "bf16"), (1032, 520, 6, 3, 2, "bf16"), (2056, 8, 4, 2, 2, "bf16"),
                                   (2048, 64, 4, 80, 2, "bf16")]:
        L = W.make_layer("toy", 603, d=d, I=I, N=N, B=B, k=k, dtype=dtype)
        out, tap = run_layer(torch, B_, L, 1, path=1)
        check_layer(oracle, L, 1, out, tap, "generic ragged d=%d I=%d" % (d, I))


def test_bias_and_padding_mask(torch, B_, oracle):
    L = W.make_layer("mid_bf16", 400, skew=True)
    mask = np.ones(L.B, np.uint8)
    mask[[1, 4, 10]] = 0
    for k0 in (2, 4):
        out, tap = run_layer(torch, B_, L, k0, bias=L.router_bias, mask=mask)
        check_layer(oracle, L, k0, out, tap, "skew+mask k0=%d" % k0, bias=L.router_bias, mask=mask)
        assert (out[[1, 4, 10]] == 0).all() and (tap["n_sel"][[1, 4, 10]] == 0).all()
    # all tokens padded: nothing active, output zero
    out, tap = run_layer(torch, B_, L, 2, mask=np.zeros(L.B, np.uint8))
    assert int(tap["n_active"][0]) == 0 and (out == 0).all()


def test_workspace_reuse_and_repeatability(torch, B_, oracle):
    big = W.make_layer("mid_bf16", 500, B=16)
    small = W.make_layer("toy", 501)
    ws = B_.new_workspace(16, big.d, big.N, big.I, big.k)
    o1, t1 = run_layer(torch, B_, big, 3, ws=ws)
    o2, t2 = run_layer(torch, B_, small, 2, ws=ws)
    o3, t3 = run_layer(torch, B_, big, 3, ws=ws)
    check_layer(oracle, big, 3, o1, t1, "reuse 1")
    check_layer(oracle, small, 2, o2, t2, "reuse 2")
    check_layer(oracle, big, 3, o3, t3, "reuse 3")
    assert np.array_equal(t1["expert_idx"], t3["expert_idx"]) and np.array_equal(t1["logits"], t3["logits"])
    # the down projection accumulates with fp32 atomics: order may differ in the last places only
    assert np.abs(o1 - o3).max() <= 1e-5 * np.abs(o1).max()


_BIG = {}


def big_layer(B_, name, seed):
    """Full-size layers are slow to draw and upload: keep the last one per name."""
    key = (name, seed)
    if _BIG.get(name, (None,))[0] != key:
        L = W.make_layer(name, seed)
        dev = {f: B_.to_device(getattr(L, f)) for f in ("x", "w_router", "w_gate", "w_up", "w_down")}
        _BIG[name] = (key, L, dev)
    return _BIG[name][1], _BIG[name][2]


@pytest.mark.parametrize("name,seeds", [("qwen3_30b", (1, 0)), ("qwen3_30b_skew", (0,))])
def test_full_size_30b_shape(torch, B_, oracle, name, seeds):
    """The configuration the benchmark times (B=16, d=2048, N=128, I=768, k=8), every output element.
    This shape runs as the single fused kernel."""
    for seed in seeds:
        L, dev = big_layer(B_, name, 2000 + seed)
        ws = B_.new_workspace(L.B, L.d, L.N, L.I, L.k)
        for k0 in ((1, 3, 5, 8) if name == "qwen3_30b" else L.k0s):
            ctx = "%s seed=%d k0=%d" % (name, seed, k0)
            out, tap = run_layer_dev(torch, B_, L, dev, k0, ws=ws, bias=L.router_bias)
            err, ref = check_layer(oracle, L, k0, out, tap, ctx, bias=L.router_bias)
            say(ctx, "T=%d sum_n_sel=%d err=%.2e" % (ref["n_active"], int(ref["n_sel"].sum()), err))


def with_inputs_of(L, B_, dev, name, seed, B=None):
    """The layer L with the token batch and the router of another seed (its expert weights kept: they do
    not enter the routing, and a full-size draw of them takes longer than everything else here)."""
    other = W.make_layer(name, seed, B=B, I=8)  # cheap: only x, the router and the bias are used
    Ln = W.Layer(**{**L.__dict__, "B": other.B, "x": other.x, "w_router": other.w_router,
                    "router_bias": other.router_bias})
    devn = dict(dev, x=B_.to_device(Ln.x), w_router=B_.to_device(Ln.w_router))
    return Ln, devn


def test_full_size_30b_eight_input_seeds(torch, B_, oracle):
    """The benchmark configuration on eight seeds of token batch and router: two draws of the expert
    weights, four draws of (x, W_router) on each; k0 = 3 and 8, every output element."""
    for wseed in (2000, 2001):
        L, dev = big_layer(B_, "qwen3_30b", wseed)
        ws = B_.new_workspace(L.B, L.d, L.N, L.I, L.k)
        for s in range(4):
            Ln, devn = with_inputs_of(L, B_, dev, "qwen3_30b", 2500 + 10 * (wseed - 2000) + s)
            for k0 in (3, 8):
                ctx = "qwen3_30b weights %d inputs %d k0=%d" % (wseed, s, k0)
                out, tap = run_layer_dev(torch, B_, Ln, devn, k0, ws=ws)
                err, ref = check_layer(oracle, Ln, k0, out, tap, ctx)
                say(ctx, "T=%d err=%.2e" % (ref["n_active"], err))


def test_full_size_30b_every_k0_and_odd_batches(torch, B_, oracle):
    """Single-kernel path at the benchmark shape: every k0 from 1 to k at B=16, and batches of 3 and 7
    tokens cut from the same layer (a workgroup then owns rows of experts with a single pair)."""
    L, dev = big_layer(B_, "qwen3_30b", 2000)
    for B in (16, 7, 3):
        ws = B_.new_workspace(B, L.d, L.N, L.I, L.k)
        x_dev = dev["x"][:B].contiguous()
        for k0 in range(1, L.k + 1):
            out, tap = B_.moe_decode(x_dev, dev["w_router"], dev["w_gate"], dev["w_up"], dev["w_down"], L.k, k0, ws,
                                     taps=True)
            torch.cuda.synchronize()
            ref = oracle.moe_decode(L.x[:B], L.w_router, L.w_gate, L.w_up, L.w_down, L.k, k0)
            ctx = "qwen3_30b B=%d k0=%d" % (B, k0)
            assert_routing_equal({n: v.cpu().numpy() for n, v in tap.items()}, ref, ctx)
            err = np.abs(out.cpu().numpy() - ref["out"]).max() / np.abs(ref["out"]).max()
            assert err <= TOL[L.dtype], "%s: %.3e" % (ctx, err)
        B_.workspace_check(ws)


@pytest.mark.parametrize("path", [2, 1])
def test_full_size_30b_shape_three_kernel_paths(torch, B_, oracle, path):
    """Same layer through the three-kernel paths (streaming / generic expert kernels)."""
    L, dev = big_layer(B_, "qwen3_30b", 2000)
    for k0 in (3, 8):
        out, tap = run_layer_dev(torch, B_, L, dev, k0, path=path)
        err, ref = check_layer(oracle, L, k0, out, tap, "path %d k0=%d" % (path, k0))
        say("path", path, "k0", k0, "T=%d err=%.2e" % (ref["n_active"], err))


def test_fused_kernel_repeatable_and_masked(torch, B_, oracle):
    """Fused path: many calls in a row on one workspace (barrier state returns to rest), a padding
    mask, an all-padding batch (no active expert: every workgroup still passes both barriers)."""
    L, dev = big_layer(B_, "qwen3_30b", 2000)
    ws = B_.new_workspace(L.B, L.d, L.N, L.I, L.k)
    first = None
    for it in range(20):
        out, tap = run_layer_dev(torch, B_, L, dev, 3, ws=ws)
        if first is None:
            first = (out, tap)
            check_layer(oracle, L, 3, out, tap, "fused repeat 0")
        else:
            assert np.array_equal(tap["expert_idx"], first[1]["expert_idx"])
            assert np.abs(out - first[0]).max() <= 1e-5 * np.abs(first[0]).max()
    mask = np.ones(L.B, np.uint8)
    mask[[0, 7, 15]] = 0
    out, tap = run_layer_dev(torch, B_, L, dev, 3, ws=ws, mask=mask)
    check_layer(oracle, L, 3, out, tap, "fused mask", mask=mask)
    out, tap = run_layer_dev(torch, B_, L, dev, 3, ws=ws, mask=np.zeros(L.B, np.uint8))
    assert int(tap["n_active"][0]) == 0 and (out == 0).all()
    for B in (1, 5, 16, 17, 32):  # both register-resident routing variants, ragged batches
        Ls = W.Layer(**{**L.__dict__, "B": B, "x": np.ascontiguousarray(np.resize(L.x, (B, L.d)))})
        devs = dict(dev, x=B_.to_device(Ls.x))
        for k0 in (2, 8):
            out, tap = run_layer_dev(torch, B_, Ls, devs, k0)
            check_layer(oracle, Ls, k0, out, tap, "fused B=%d k0=%d" % (B, k0))


def test_full_size_30b_batch_sweep(torch, B_, oracle):
    L0 = W.make_layer("qwen3_30b", 2100, B=160)
    dev_w = {f: B_.to_device(getattr(L0, f)) for f in ("w_router", "w_gate", "w_up", "w_down")}
    # up to 32: single kernel with x resident; 64, 128: single kernel with per-workgroup staging;
    # 160: router kernel and the two stage kernels
    for B in (1, 2, 4, 8, 16, 32, 64, 128, 160):
        L = W.Layer(**{**L0.__dict__, "B": B, "x": np.ascontiguousarray(L0.x[:B])})
        dev = dict(dev_w, x=B_.to_device(L.x))
        for k0 in (3, 5, 8):
            ctx = "30b-shape B=%d k0=%d" % (B, k0)
            out, tap = run_layer_dev(torch, B_, L, dev, k0)
            err, ref = check_layer(oracle, L, k0, out, tap, ctx)
            say(ctx, "T=%d err=%.2e" % (ref["n_active"], err))
    # ragged batches through the kernel with per-workgroup staging: a last token group that is not full,
    # padded tokens, a router bias, Phase 2 with and without rounds
    rng = np.random.Generator(np.random.PCG64(77))
    bias = (rng.standard_normal(L0.N) * 0.7).astype(np.float32)
    for B in (33, 50, 100, 127):
        L = W.Layer(**{**L0.__dict__, "B": B, "x": np.ascontiguousarray(L0.x[160 - B:])})
        dev = dict(dev_w, x=B_.to_device(L.x))
        mask = (rng.integers(0, 5, size=B) != 0).astype(np.uint8)
        for k0 in (3, 8):
            ctx = "30b-shape ragged B=%d k0=%d, mask and bias" % (B, k0)
            out, tap = run_layer_dev(torch, B_, L, dev, k0, bias=bias, mask=mask)
            err, ref = check_layer(oracle, L, k0, out, tap, ctx, bias=bias, mask=mask)
            assert (out[mask == 0] == 0).all()
            say(ctx, "T=%d live=%d err=%.2e" % (ref["n_active"], int(mask.sum()), err))


def test_full_size_235b_shape(torch, B_, oracle):
    _BIG.clear()
    L = W.make_layer("qwen3_235b", 3000)
    dev = {f: B_.to_device(getattr(L, f)) for f in ("x", "w_router", "w_gate", "w_up", "w_down")}
    for k0 in range(1, L.k + 1):  # every k0, on two seeds of token batch and router
        for s in (0, 1):
            Ln, devn = (L, dev) if s == 0 else with_inputs_of(L, B_, dev, "qwen3_235b", 3100)
            ctx = "qwen3_235b inputs %d k0=%d" % (s, k0)
            out, tap = run_layer_dev(torch, B_, Ln, devn, k0)
            err, ref = check_layer(oracle, Ln, k0, out, tap, ctx)
            say(ctx, "T=%d err=%.2e" % (ref["n_active"], err))
    for k0 in (3, 8):  # the three-kernel path with the streaming expert kernels
        ctx = "qwen3_235b path=2 k0=%d" % k0
        out, tap = run_layer_dev(torch, B_, L, dev, k0, path=2)
        err, ref = check_layer(oracle, L, k0, out, tap, ctx)
        say(ctx, "T=%d err=%.2e" % (ref["n_active"], err))
    # a larger batch on the same weights: the single kernel with per-workgroup staging (vectors of
    # 8 KB leave room for about a dozen per workgroup, so pieces occur)
    L48 = W.make_layer("qwen3_235b", 3001, B=48, N=1, I=8)  # only its x is used
    Lb = W.Layer(**{**L.__dict__, "B": 48, "x": L48.x})
    devb = dict(dev, x=B_.to_device(Lb.x))
    out, tap = run_layer_dev(torch, B_, Lb, devb, 3)
    err, ref = check_layer(oracle, Lb, 3, out, tap, "qwen3_235b B=48 k0=3")
    say("qwen3_235b B=48 k0=3 T=%d err=%.2e" % (ref["n_active"], err))
    # the same batch through the matrix-core expert stages (this shape: 12 and 16 units per expert, 64 and
    # 24 slabs per unit); the oracle's result of the run above serves again
    out4, tap4 = run_layer_dev(torch, B_, Lb, devb, 3, path=4)
    assert np.array_equal(tap4["expert_idx"], tap["expert_idx"]) and np.array_equal(tap4["logits"], tap["logits"])
    err4 = np.abs(out4.astype(np.float64) - ref["out"]).max() / np.abs(ref["out"]).max()
    say("qwen3_235b B=48 k0=3 matrix-core stages err=%.2e" % err4)
    assert err4 <= TOL[Lb.dtype]


# ---- general OEA (Algorithm 2): top-p cut of the baseline, k_max, rank window max_p

def route_general_gpu(torch, B_, lg, k0, p, k_max, max_p, mask=None):
    res = B_.oea_route_general(torch.from_numpy(lg).cuda(), k0, p, k_max, max_p,
                               token_mask=None if mask is None else torch.from_numpy(mask).cuda())
    torch.cuda.synchronize()
    return {n: v.cpu().numpy() for n, v in res.items()}


def top_p_is_clear(lg, k0, p, margin=1e-9):
    """True if no token's sorted cumulative softmax mass comes within `margin` of p inside its k0
    best experts: then the top-p decision cannot depend on the summation order."""
    if p >= 1.0:
        return True
    l = lg.astype(np.float64)
    r = np.exp(l - l.max(axis=1, keepdims=True))
    r /= r.sum(axis=1, keepdims=True)
    cum = np.cumsum(-np.sort(-r, axis=1), axis=1)[:, :k0]
    return bool((np.abs(cum - p) > margin).all())


GENERAL_CASES = [(B, N, k0, p, k_max, max_p, kind, seed)
                 for (B, N) in [(16, 128), (4, 16), (33, 64), (7, 200), (130, 100), (1, 128)]
                 for (k0, k_max) in [(1, 4), (3, 8), (8, 8), (6, 4), (2, 12)]
                 for p in (1.0, 0.9, 0.5, 0.2)
                 for max_p in ("N", 32, 5)
                 for kind in ("gaussian", "skew", "ties", "wide")
                 for seed in (0,)]


def test_route_general_bit_exact(torch, B_, oracle):
    n = skipped = 0
    for (B, N, k0, p, k_max, max_p, kind, seed) in GENERAL_CASES:
        if k0 > N or k_max > N:
            continue
        mp = N if max_p == "N" else min(max_p, N)
        lg = W.make_logits(B, N, 700 + seed, kind)
        if not top_p_is_clear(lg, k0, p):
            skipped += 1
            continue
        mask = None
        if B >= 4 and seed == 0 and kind == "skew":
            mask = np.ones(B, np.uint8)
            mask[1::3] = 0
        ctx = "general B=%d N=%d k0=%d p=%g k_max=%d max_p=%d kind=%s" % (B, N, k0, p, k_max, mp, kind)
        got = route_general_gpu(torch, B_, lg, k0, p, k_max, mp, mask)
        ref = oracle.route_general(lg, k0, p, k_max, mp, token_mask=mask)
        assert np.array_equal(got["n_base"], ref["n_base"]), ctx
        assert_routing_equal(got, ref, ctx)
        n += 1
    say("general routing cases checked: %d, skipped as ambiguous: %d" % (n, skipped))
    assert n > 1000 and skipped < n // 20


def test_route_general_reduces_to_algorithm_1(torch, B_):
    for (B, N, k, k0) in [(16, 128, 8, 3), (33, 64, 6, 6), (5, 512, 32, 7), (200, 130, 8, 1)]:
        lg = W.make_logits(B, N, 42, "gaussian")
        a = route_gpu(torch, B_, lg, k, k0)
        g = route_general_gpu(torch, B_, lg, k0, 1.0, k, N)
        for f in ("expert_idx", "n_sel", "active_list", "n_active"):
            assert np.array_equal(a[f], g[f]), (B, N, k, k0, f)
        assert np.array_equal(a["gate_w"], g["gate_w"]) or np.abs(a["gate_w"] - g["gate_w"]).max() <= 1e-6
        assert (g["n_base"] == k0).all()


def test_layer_general_oea(torch, B_, oracle):
    """The whole layer under Algorithm 2 (top-p cut and rank window), three-kernel path; above B = 128
    the router and the routing run as four kernels over many workgroups."""
    for name, B, k0, p, max_p in (("mid_bf16", None, 3, 0.2, None), ("mid_bf16", None, 4, None, 6),
                                  ("qwen3_30b", None, 3, 0.1, 24),
                                  ("mid_bf16", 200, 3, 0.2, None), ("mid_bf16", 300, 4, None, 6),
                                  ("mid_bf16", 150, 3, 0.15, 8), ("mid_bf16", 1024, 2, 0.3, 5),
                                  ("qwen3_30b", 160, 3, 0.1, 24)):
        L = W.make_layer(name, 11, B=B)
        dev = {f: B_.to_device(getattr(L, f)) for f in ("x", "w_router", "w_gate", "w_up", "w_down")}
        ws = B_.new_workspace(L.B, L.d, L.N, L.I, L.k)
        out, tap = B_.moe_decode(dev["x"], dev["w_router"], dev["w_gate"], dev["w_up"], dev["w_down"], L.k, k0, ws,
                                 taps=True, top_p=p, max_p=max_p)
        torch.cuda.synchronize()
        tap = {n: v.cpu().numpy() for n, v in tap.items()}
        pp, mp = (1.0 if p is None else p), (L.N if max_p is None else max_p)
        ctx = "layer general %s B=%d k0=%d p=%s max_p=%s" % (name, L.B, k0, p, max_p)
        assert top_p_is_clear(tap["logits"], k0, pp), ctx
        ref = oracle.route_general(tap["logits"], k0, pp, L.k, mp)
        assert_routing_equal(tap, ref, ctx)
        if p is not None:
            assert (ref["n_base"] < k0).any(), "the top-p cut should bite in this case"
        ref_out = oracle.moe_combine(L.x, L.w_gate, L.w_up, L.w_down, ref["expert_idx"], ref["gate_w"])
        err = np.abs(out.cpu().numpy().astype(np.float64) - ref_out).max() / np.abs(ref_out).max()
        say("%s: T=%d, max|d|/max|ref| = %.2e" % (ctx, ref["n_active"], err))
        assert err <= TOL[L.dtype], ctx


def test_layer_general_oea_single_kernel(torch, B_, oracle):
    """Algorithm 2 inside the single-kernel layer (30B shape, both kernel variants: B <= 32 and
    larger): top-p cut, rank window, both, with a padding mask, for several batch sizes; the
    three-kernel path must route identically."""
    L0, dev0 = big_layer(B_, "qwen3_30b", 2000)
    L32 = W.make_layer("qwen3_30b", 2100, B=32, I=8)  # token vectors only (the expert weights are L0's)
    xs = {b: np.ascontiguousarray(L0.x[:b]) for b in (1, 5, 16)}
    xs[32] = np.ascontiguousarray(L32.x)
    for b in (50, 64, 128):  # the kernel variant for larger batches: token groups, baselines parked between the phases
        xs[b] = np.ascontiguousarray(W.make_layer("qwen3_30b", 2100 + b, B=b, I=8).x)
    cases = [(16, 3, 0.1, None, False), (16, 3, None, 8, False), (16, 3, 0.1, 24, False), (16, 4, 0.08, 12, True),
             (16, 8, 0.3, None, False), (16, 2, None, 3, False), (1, 3, 0.1, 6, False), (5, 3, 0.12, 10, True),
             (32, 3, 0.1, 16, True), (32, 5, None, 6, False),
             (50, 3, 0.1, 12, True), (64, 3, 0.1, None, False), (64, 4, None, 8, True), (128, 3, 0.12, 24, False),
             (128, 2, None, 5, True)]
    for b, k0, p, max_p, masked in cases:
        L = W.Layer(**{**L0.__dict__, "x": xs[b], "B": b})
        dev = dict(dev0, x=B_.to_device(L.x))
        mask = None
        if masked:
            mask = np.ones(b, np.uint8)
            mask[1::3] = 0
        dmask = None if mask is None else torch.from_numpy(mask).cuda()
        ws = B_.new_workspace(L.B, L.d, L.N, L.I, L.k)
        taps = {}
        for path in (None, 2):
            out, tap = B_.moe_decode(dev["x"], dev["w_router"], dev["w_gate"], dev["w_up"], dev["w_down"], L.k, k0,
                                     ws, taps=True, top_p=p, max_p=max_p, token_mask=dmask, kernel_path=path)
            torch.cuda.synchronize()
            B_.workspace_check(ws)
            taps[path] = ({n: v.cpu().numpy() for n, v in tap.items()}, out.cpu().numpy().astype(np.float64))
        tap, got = taps[None]
        pp, mp = (1.0 if p is None else p), (L.N if max_p is None else max_p)
        ctx = "single-kernel general B=%d k0=%d p=%s max_p=%s mask=%s" % (b, k0, p, max_p, masked)
        assert top_p_is_clear(tap["logits"], k0, pp), ctx
        ref = oracle.route_general(tap["logits"], k0, pp, L.k, mp, token_mask=mask)
        assert_routing_equal(tap, ref, ctx)
        assert_routing_equal(taps[2][0], ref, ctx + " (three kernels)")
        ref_out = oracle.moe_combine(L.x, L.w_gate, L.w_up, L.w_down, ref["expert_idx"], ref["gate_w"])
        err = np.abs(got - ref_out).max() / np.abs(ref_out).max()
        say("%s: T=%d, mean |S_i| %.2f, max|d|/max|ref| = %.2e" % (ctx, ref["n_active"], ref["n_sel"].mean(), err))
        assert err <= TOL[L.dtype], ctx


# ---- many decode positions in one launch

def test_route_batched_positions(torch, B_, oracle):
    for (L, B, N, k, k0, masked) in [(64, 16, 128, 8, 3, False), (37, 5, 200, 12, 6, True), (9, 70, 64, 6, 2, True),
                                      (300, 16, 128, 8, 8, False), (3, 1, 16, 4, 1, False)]:
        lg = np.stack([W.make_logits(B, N, 300 + l, "gaussian" if l % 3 else "ties") for l in range(L)])
        mask = None
        if masked:
            mask = (np.arange(L * B).reshape(L, B) % 4 != 1).astype(np.uint8)
        res = B_.oea_route_batched(torch.from_numpy(lg).cuda(), k, k0,
                                   token_mask=None if mask is None else torch.from_numpy(mask).cuda())
        torch.cuda.synchronize()
        res = {n: v.cpu().numpy() for n, v in res.items()}
        for l in range(L):
            ref = oracle.route(lg[l], k, k0, token_mask=None if mask is None else mask[l])
            got = {n: v[l] for n, v in res.items()}
            got["n_active"] = np.array([got["n_active"]])
            assert_routing_equal(got, ref, "batched L=%d B=%d N=%d k=%d k0=%d position %d" % (L, B, N, k, k0, l))
    # throughput of the routing step alone at the Qwen3-30B-A3B shape (reported, not asserted)
    L = 4096
    lg = torch.randn((L, 16, 128), device="cuda", dtype=torch.float32)
    B_.oea_route_batched(lg, 8, 3)
    torch.cuda.synchronize()
    e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    e0.record()
    for _ in range(10):
        B_.oea_route_batched(lg, 8, 3)
    e1.record()
    torch.cuda.synchronize()
    us = e0.elapsed_time(e1) * 1e3 / 10
    say("oea_route_batched: %d positions of B=16, N=128 in %.1f us (%.1f M positions/s)" % (L, us, L / us))


LANE_CASES = [  # (L, B, N, k, k0, kind of logits, masked): at and above the sizes where a lane takes a token
    (2560, 16, 128, 8, 3, "gaussian", False), (2563, 16, 128, 8, 8, "ties", True), (2595, 15, 128, 8, 1, "constant", False),
    (2600, 16, 128, 7, 2, "signed_zero", True), (2560, 16, 64, 8, 5, "denormal", False), (2680, 13, 36, 6, 4, "minus_inf", False),
    (2560, 16, 128, 8, 3, "minus_inf", True), (2560, 16, 100, 8, 6, "plus_inf", False), (512, 64, 128, 8, 7, "skew", True),
    (515, 63, 68, 8, 4, "gaussian", False), (513, 33, 4, 4, 2, "ties", True), (10240, 1, 128, 8, 3, "ties", False),
    (6144, 2, 4, 1, 1, "gaussian", True), (4096, 4, 60, 5, 3, "wide", False), (3840, 16, 128, 16, 16, "ties", False),
    (3841, 16, 128, 12, 6, "gaussian", True), (768, 40, 64, 10, 3, "minus_inf", False), (3840, 16, 96, 9, 4, "constant", True),
    (2560, 16, 128, 8, 3, "nan", False), (3840, 16, 64, 12, 5, "nan", True)]


@pytest.mark.parametrize("case", LANE_CASES, ids=lambda c: "L%d-B%d-N%d-k%d-k0%d-%s%s" % (c[:6] + ("-masked" if c[6] else "",)))
def test_route_batched_lane_per_token(torch, B_, oracle, case):
    """The routing kernel for many positions (a lane per token, 64 / B positions per wavefront): remainders of
    positions and tokens, ragged expert counts, lists of 8 and 16, ties at every limit, infinities, padding."""
    L, B, N, k, k0, kind, masked = case
    rng = np.random.default_rng(L * 31 + N)
    if kind == "nan":
        lg = rng.standard_normal((L, B, N), dtype=np.float32)
        lg[rng.random((L, B, N)) < 0.2] = np.nan
    elif kind in ("minus_inf", "plus_inf"):
        # experts switched off by the lowest values there are, in every second position down to fewer than k live ones
        lg = rng.standard_normal((L, B, N), dtype=np.float32)
        off = rng.random((L, 1, N)) < np.where(np.arange(L) % 2, 0.95, 0.3)[:, None, None]
        lg = np.where(off, np.float32(-np.inf) if kind == "minus_inf" else np.finfo(np.float32).min, lg)
        lg[:, :, 1] = 0.5  # one expert is always on, so that the weights are numbers
        if kind == "plus_inf":
            lg[::3, :, 2] = np.inf
            lg[::6, :, 5:15:2] = np.inf
    else:
        lg = W.make_logits(L * B, N, 4000 + k0, kind).reshape(L, B, N)
    mask = (rng.random((L, B)) > 0.3).astype(np.uint8) if masked else None
    if masked:
        mask[L // 2] = 0  # a position of padding only
    res = B_.oea_route_batched(torch.from_numpy(lg).cuda(), k, k0,
                               token_mask=None if mask is None else torch.from_numpy(mask).cuda())
    torch.cuda.synchronize()
    res = {n: v.cpu().numpy() for n, v in res.items()}
    if kind == "nan":  # which experts is unspecified; every index is one
        assert res["expert_idx"].min() >= -1 and res["expert_idx"].max() < N
        assert res["active_list"].min() >= -1 and res["active_list"].max() < N
        assert res["n_sel"].min() >= 0 and res["n_sel"].max() <= k and res["n_active"].max() <= N
        return
    for l in range(L):
        ref = oracle.route(lg[l], k, k0, token_mask=None if mask is None else mask[l])
        for name in ("expert_idx", "n_sel", "active_list"):
            assert np.array_equal(res[name][l], ref[name]), (name, l, res[name][l], ref[name])
        assert int(res["n_active"][l]) == int(ref["n_active"])
        if kind != "plus_inf":  # (the softmax of an infinite logit is not a number)
            assert np.abs(res["gate_w"][l] - ref["gate_w"]).max() <= 1e-6, l


NAN_CASES = [  # (L, B, N, k, k0, share of NaN logits in every second position, their bit patterns)
    (2560, 16, 128, 8, 3, 0.2, (0x7FC00000,)), (2564, 16, 128, 8, 8, 0.01, (0x7FC00000, 0xFFC00000)),
    (2560, 16, 128, 7, 1, 0.9, (0x7FC00000, 0xFFC00000, 0x7F800001, 0xFF800001, 0x7FFFFFFF, 0xFFFFFFFE)),
    (2600, 15, 60, 8, 4, 0.95, (0xFFC00000,)), (3840, 16, 96, 12, 5, 0.5, (0x7FC00000, 0xFFC12345)),
    (6144, 2, 4, 4, 4, 0.3, (0x7FC00000, 0xFFC00000)), (10240, 1, 64, 8, 2, 0.5, (0x7FC00000, 0xFFC00000)),
    (768, 64, 64, 16, 16, 0.3, (0x7FD00000, 0xFFC00000))]


@pytest.mark.parametrize("case", NAN_CASES, ids=lambda c: "L%d-B%d-N%d-k%d-k0%d-%.2f" % c[:6])
def test_route_batched_logits_that_are_not_numbers(torch, B_, case):
    """Logits that are not numbers give the same routing in a launch of many positions (a lane per token) as in
    launches of few (a row of lanes per token): ids distinct, at most k0 per token in the union, neighbours and other
    positions untouched, and no finite weights for a token that has selected a NaN."""
    L, B, N, k, k0, share, patterns = case
    rng = np.random.default_rng(L + N + k)
    lg = rng.standard_normal((L, B, N), dtype=np.float32)
    lg[rng.random((L, B, N)) < 0.1] = -np.inf
    lg[1::7] = np.round(lg[1::7])  # ties
    lg[5::8, :, :k0] = np.inf      # as many as a token keeps
    bad = rng.random((L, B, N)) < share
    bad[::2] = False
    bad[1::8, ::2] = False  # tokens without a NaN beside tokens with one
    bad[3::8, 0] = True     # a token of NaNs alone
    bits = lg.view(np.uint32)
    bits[bad] = rng.choice(np.array(patterns, np.uint32), int(bad.sum()))
    mask = (rng.random((L, B)) > 0.2).astype(np.uint8)
    dl, dm = torch.from_numpy(lg).cuda(), torch.from_numpy(mask).cuda()
    got = {n: v.cpu().numpy() for n, v in B_.oea_route_batched(dl, k, k0, token_mask=dm).items()}
    few = 200  # below every size at which a lane takes a token
    parts = [B_.oea_route_batched(dl[l:l + few], k, k0, token_mask=dm[l:l + few]) for l in range(0, L, few)]
    ref = {n: np.concatenate([p[n].cpu().numpy() for p in parts]) for n in got}
    for name in ("n_active", "active_list", "n_sel", "expert_idx"):
        differ = np.nonzero((got[name] != ref[name]).reshape(L, -1).any(1))[0]
        assert differ.size == 0, (name, differ[:5], got[name][differ[0]], ref[name][differ[0]])
    assert np.array_equal(got["gate_w"], ref["gate_w"], equal_nan=True)
    chosen = np.take_along_axis(lg, np.maximum(got["expert_idx"], 0), 2)
    used = got["expert_idx"] >= 0
    hit = (np.isnan(chosen) & used).any(2)
    assert hit.any() and np.isnan(got["gate_w"][hit][used[hit]]).all()


def test_single_kernel_routing_many_batches(torch, B_, oracle):
    """The routing inside the single-kernel layer (rows of 16 lanes, hand-scheduled selection round,
    bookkeeping on the wavefronts without tokens) over many token batches: B = 1..32, every k0, with
    and without a padding mask, compared with the oracle on the logits the kernel computed.  The
    expert weights do not enter the routing: random ones drawn on the device."""
    d, N, I, k = 2048, 128, 768, 8
    g = torch.Generator(device="cuda")
    g.manual_seed(5)
    wts = tuple(torch.randn(sh, generator=g, device="cuda", dtype=torch.float32).mul_(0.02).to(torch.bfloat16)
                for sh in ((N, I, d), (N, I, d), (N, d, I)))
    rng = np.random.default_rng(123)
    n = 0
    for b in (1, 2, 3, 5, 8, 11, 16, 24, 32):
        ws = B_.new_workspace(b, d, N, I, k)
        for seed in range(6):
            L = W.make_layer("qwen3_30b", 50000 + 100 * b + seed, B=b, I=8)  # token vectors and router
            x, wr = B_.to_device(L.x), B_.to_device(L.w_router)
            mask = None
            if seed % 3 == 2 and b > 1:
                mask = (rng.random(b) > 0.3).astype(np.uint8)
                mask[0] = 1
            dm = None if mask is None else torch.from_numpy(mask).cuda()
            for k0 in range(1, 9):
                _, tap = B_.moe_decode(x, wr, *wts, k, k0, ws, taps=True, token_mask=dm)
                torch.cuda.synchronize()
                tap = {m: v.cpu().numpy() for m, v in tap.items()}
                assert_routing_equal(tap, oracle.route(tap["logits"], k, k0, token_mask=mask),
                                     "single-kernel routing B=%d seed=%d k0=%d" % (b, seed, k0))
                n += 1
        B_.workspace_check(ws)
    say("single-kernel routing cases checked:", n)


@pytest.mark.parametrize("path", [2, 3])
def test_three_kernel_paths_small_batches(torch, B_, oracle, path):
    """The router + routing kernel with 16 wavefronts: for few tokens most of them hold no token row
    and do the per-expert bookkeeping beside the selection rounds (B = 1, 5, 8: one row per
    wavefront; B = 11: four rows per wavefront, three busy wavefronts)."""
    L0, dev0 = big_layer(B_, "qwen3_30b", 2000)
    for b in (1, 5, 8, 11):
        L = W.Layer(**{**L0.__dict__, "x": np.ascontiguousarray(L0.x[:b]), "B": b})
        dev = dict(dev0, x=B_.to_device(L.x))
        for k0 in (3, 8):
            out, tap = run_layer_dev(torch, B_, L, dev, k0, path=path)
            err, ref = check_layer(oracle, L, k0, out, tap, "path %d B=%d k0=%d" % (path, b, k0))
            say("path", path, "B", b, "k0", k0, "T=%d err=%.2e" % (ref["n_active"], err))


# ---- larger batches: the expert stages as separate kernels

def test_stage_kernels_at_b16(torch, B_, oracle):
    """Kernel path 3 runs the stage kernels also where the fused kernel would apply."""
    L = W.make_layer("qwen3_30b", 77)
    dev = {f: B_.to_device(getattr(L, f)) for f in ("x", "w_router", "w_gate", "w_up", "w_down")}
    for k0 in (1, 3, 8):
        out, tap = run_layer_dev(torch, B_, L, dev, k0, path=3)
        err, ref = check_layer(oracle, L, k0, out, tap, "stage kernels B=16 k0=%d" % k0)
        say("stage kernels B=16 k0=%d T=%d err=%.2e" % (k0, ref["n_active"], err))


def test_many_tokens_per_expert(torch, B_, oracle):
    """B=64 near-identical tokens: every active expert serves all of them, so a workgroup's pair list
    exceeds its LDS share and is walked in pieces."""
    L0 = W.make_layer("qwen3_30b", 78, B=64)
    x = np.repeat(L0.x[:1], 64, axis=0).copy()
    x[1::2] = L0.x[1:2]  # two distinct tokens, alternating
    L = W.Layer(**{**L0.__dict__, "x": np.ascontiguousarray(x)})
    dev = {f: B_.to_device(getattr(L, f)) for f in ("x", "w_router", "w_gate", "w_up", "w_down")}
    for path in (0, 3):  # the single kernel for larger batches, and the separate stage kernels
        for k0 in (2, 8):
            out, tap = run_layer_dev(torch, B_, L, dev, k0, path=path)
            err, ref = check_layer(oracle, L, k0, out, tap, "B=64 duplicated tokens k0=%d path %d" % (k0, path))
            cnt = np.bincount(ref["expert_idx"][ref["expert_idx"] >= 0], minlength=L.N)
            say("B=64 duplicated tokens k0=%d path %d: T=%d, most pairs on one expert %d, err=%.2e"
                % (k0, path, ref["n_active"], cnt.max(), err))
            assert cnt.max() >= 32


def test_matrix_core_stages(torch, B_, oracle):
    """The expert stages on the matrix cores (kernel path 4, and the automatic choice, which takes them above B=128 at
    these sizes): batches in which an expert serves a few tokens (one partly filled group of 16), many (several groups), and
    more than 64; the skewed workload; padding; the deterministic combine.  (More tokens than the 128 of a pass:
    test_matrix_core_granules.)"""
    L0 = W.make_layer("qwen3_30b", 2100, B=160)
    dev_w = {f: B_.to_device(getattr(L0, f)) for f in ("w_router", "w_gate", "w_up", "w_down")}

    def case(ctx, x, k0, path, bias=None, mask=None, min_pairs=0):
        L = W.Layer(**{**L0.__dict__, "B": x.shape[0], "x": np.ascontiguousarray(x)})
        dev = dict(dev_w, x=B_.to_device(L.x))
        say(ctx)
        out, tap = run_layer_dev(torch, B_, L, dev, k0, bias=bias, mask=mask, path=path)
        err, ref = check_layer(oracle, L, k0, out, tap, ctx, bias=bias, mask=mask)
        cnt = np.bincount(ref["expert_idx"][ref["expert_idx"] >= 0], minlength=L.N)
        say("   T=%d, most pairs on one expert %d, err=%.2e" % (ref["n_active"], cnt.max(), err))
        assert cnt.max() >= min_pairs
        return L, dev

    for k0 in (3, 5, 8):
        case("matrix cores B=128 k0=%d" % k0, L0.x[:128], k0, 4)
    for B in (1, 5, 16, 37):
        case("matrix cores B=%d k0=3" % B, L0.x[:B], 3, 4)
    # two distinct tokens, alternating: every active expert serves 32 of the 64 tokens
    x = np.repeat(L0.x[:1], 64, axis=0).copy()
    x[1::2] = L0.x[1:2]
    for k0 in (2, 8):
        case("matrix cores B=64 duplicated tokens k0=%d" % k0, x, k0, 4, min_pairs=32)
    # the skewed-popularity workload: few experts, up to all 16 tokens on one
    Ls = W.make_layer("qwen3_30b_skew", 2000, I=8)  # its token batch, router and bias; expert weights of L0
    Lsk = W.Layer(**{**L0.__dict__, "B": Ls.B, "x": Ls.x, "w_router": Ls.w_router})
    devs = dict(dev_w, x=B_.to_device(Lsk.x), w_router=B_.to_device(Lsk.w_router))
    for k0 in (2, 4):
        out, tap = run_layer_dev(torch, B_, Lsk, devs, k0, bias=Ls.router_bias, path=4)
        err, ref = check_layer(oracle, Lsk, k0, out, tap, "matrix cores skew k0=%d" % k0, bias=Ls.router_bias)
        say("matrix cores skew k0=%d: T=%d err=%.2e" % (k0, ref["n_active"], err))
    # automatic choice above B=128: three distinct tokens in turn, so experts serve about 85 of the 256
    # tokens (six groups of 16, the last one ragged); padding mask
    x = np.ascontiguousarray(L0.x[np.arange(256) % 3])
    mask = np.ones(256, np.uint8)
    mask[[0, 100, 255]] = 0
    L, dev = case("matrix cores B=256, three distinct tokens, automatic path, mask", x, 3, None, mask=mask, min_pairs=65)
    # small shapes: both stages on the matrix cores (several experts per workgroup, more workgroups than units)
    for (d, I, N, B, k) in [(512, 256, 6, 200, 3), (256, 256, 3, 40, 2), (256, 128, 8, 40, 2), (1024, 512, 20, 300, 4)]:
        Lt = W.make_layer("toy", 640, d=d, I=I, N=N, B=B, k=k, dtype="bf16")
        for k0 in (1, k):
            for path in (4, None):
                out, tap = run_layer(torch, B_, Lt, k0, path=path)
                check_layer(oracle, Lt, k0, out, tap, "matrix cores d=%d I=%d N=%d B=%d k0=%d path %s" % (d, I, N, B, k0, path))
    # a ragged batch above 128 with a router bias and padded tokens, Phase 2 with and without rounds (the
    # router and the routing then run as four kernels over many workgroups)
    rng = np.random.Generator(np.random.PCG64(78))
    bias = (rng.standard_normal(L0.N) * 0.7).astype(np.float32)
    x = np.ascontiguousarray(np.concatenate([L0.x, L0.x[:43][::-1]]))  # 203 tokens
    mask = (rng.integers(0, 6, size=x.shape[0]) != 0).astype(np.uint8)
    for k0 in (3, 8):
        case("matrix cores B=203 k0=%d, bias and mask" % k0, x, k0, None, bias=bias, mask=mask)
    # deterministic combine through the same stages: one row per pair, bit-identical from call to call
    ws = B_.new_workspace(L.B, L.d, L.N, L.I, L.k, deterministic=True)
    first = None
    for it in range(4):
        out, tap = B_.moe_decode(dev["x"], dev["w_router"], dev["w_gate"], dev["w_up"], dev["w_down"], L.k, 3, ws,
                                 taps=True, deterministic=True)
        torch.cuda.synchronize()
        o = out.cpu().numpy()
        if first is None:
            first = o
            check_layer(oracle, L, 3, o, {n: v.cpu().numpy() for n, v in tap.items()}, "matrix cores deterministic B=256")
        else:
            assert np.array_equal(o.view(np.uint32), first.view(np.uint32)), "call %d differs" % it


# ---- capture into a HIP graph

def test_graph_capture_and_replay(torch, B_, oracle):
    """Two layers (fused single-kernel path) captured into one graph; every replay, with eager work in
    between, must reproduce the eager result."""
    L = W.make_layer("qwen3_30b", 91, B=8)
    dev = {f: B_.to_device(getattr(L, f)) for f in ("x", "w_router", "w_gate", "w_up", "w_down")}
    ws = B_.new_workspace(L.B, L.d, L.N, L.I, L.k)
    out_a = torch.empty((L.B, L.d), dtype=torch.float32, device="cuda")
    out_b = torch.empty_like(out_a)

    def two_layers():
        B_.moe_decode(dev["x"], dev["w_router"], dev["w_gate"], dev["w_up"], dev["w_down"], L.k, 2, ws, out=out_a)
        B_.moe_decode(dev["x"], dev["w_router"], dev["w_gate"], dev["w_up"], dev["w_down"], L.k, 8, ws, out=out_b)

    two_layers()
    torch.cuda.synchronize()
    eager_a, eager_b = out_a.cpu().numpy().copy(), out_b.cpu().numpy().copy()
    ref = oracle.moe_decode(L.x, L.w_router, L.w_gate, L.w_up, L.w_down, L.k, 2)
    assert np.abs(eager_a - ref["out"]).max() / np.abs(ref["out"]).max() <= TOL[L.dtype]
    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    g = torch.cuda.CUDAGraph()
    with torch.cuda.stream(s):
        with torch.cuda.graph(g, stream=s):
            two_layers()
    torch.cuda.synchronize()
    for rep in range(4):
        out_a.fill_(7.0)  # eager work between the replays: poison the outputs, run an unrelated layer
        out_b.fill_(7.0)
        B_.moe_decode(dev["x"], dev["w_router"], dev["w_gate"], dev["w_up"], dev["w_down"], L.k, 5,
                      B_.new_workspace(L.B, L.d, L.N, L.I, L.k))
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        for got, want, name in ((out_a, eager_a, "k0=2"), (out_b, eager_b, "k0=8")):
            err = np.abs(got.cpu().numpy() - want).max() / np.abs(want).max()
            assert err <= 1e-5, "replay %d %s: %.2e" % (rep, name, err)
    say("graph replays match the eager result")


def test_graph_capture_large_batch(torch, B_, oracle):
    """A batch above 128 (router and routing as four kernels, expert stages on the matrix cores: six
    kernels per layer) captured into a graph; every replay must reproduce the eager routing, and the
    deterministic combine the eager output bit for bit."""
    L = W.make_layer("toy", 92, d=512, I=256, N=12, B=200, k=4, dtype="bf16")
    dev = {f: B_.to_device(getattr(L, f)) for f in ("x", "w_router", "w_gate", "w_up", "w_down")}
    ws = B_.new_workspace(L.B, L.d, L.N, L.I, L.k, deterministic=True)
    out = torch.empty((L.B, L.d), dtype=torch.float32, device="cuda")

    def layer():
        B_.moe_decode(dev["x"], dev["w_router"], dev["w_gate"], dev["w_up"], dev["w_down"], L.k, 2, ws, out=out,
                      deterministic=True)

    layer()
    torch.cuda.synchronize()
    eager = out.cpu().numpy().copy()
    ref = oracle.moe_decode(L.x, L.w_router, L.w_gate, L.w_up, L.w_down, L.k, 2)
    assert np.abs(eager - ref["out"]).max() / np.abs(ref["out"]).max() <= TOL[L.dtype]
    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    g = torch.cuda.CUDAGraph()
    with torch.cuda.stream(s):
        with torch.cuda.graph(g, stream=s):
            layer()
    torch.cuda.synchronize()
    for rep in range(4):
        out.fill_(7.0)
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        assert np.array_equal(out.cpu().numpy().view(np.uint32), eager.view(np.uint32)), "replay %d" % rep
    B_.workspace_check(ws)
    say("graph replays of a large batch match the eager result bit for bit")


def test_unprepared_workspace_is_reported_at_once(torch, B_, oracle):
    """A layer on a workspace that oea_workspace_init never saw (or that was overwritten since) does not
    spin: its kernels return early and oea_workspace_check names the cause.  Both the single-kernel
    path and the three-kernel path; afterwards the prepared workspace works."""
    import time
    for name, B in (("qwen3_30b", 4), ("mid_bf16", None)):
        L = W.make_layer(name, 95, B=B)
        dev = {f: B_.to_device(getattr(L, f)) for f in ("x", "w_router", "w_gate", "w_up", "w_down")}
        n = B_.workspace_bytes(L.B, L.d, L.N, L.I, L.k)
        ws = torch.randint(0, 255, (n,), dtype=torch.uint8, device="cuda")  # never prepared: arbitrary control words
        args = (dev["x"], dev["w_router"], dev["w_gate"], dev["w_up"], dev["w_down"], L.k, 2, ws)
        say("%s: layer on an unprepared workspace" % name)
        t0 = time.perf_counter()
        B_.moe_decode(*args)
        with pytest.raises(B_.OeaError) as err:
            B_.workspace_check(ws)
        assert err.value.code == B_.STATUS["OEA_ERR_WORKSPACE_STATE"]
        assert time.perf_counter() - t0 < 0.5, "the kernels must not wait out their poll limit"
        # prepared, used, then overwritten by the caller
        B_.workspace_init(ws)
        good = B_.moe_decode(*args).cpu().numpy()
        B_.workspace_check(ws)
        ref = oracle.moe_decode(L.x, L.w_router, L.w_gate, L.w_up, L.w_down, L.k, 2)
        assert np.abs(good - ref["out"]).max() / np.abs(ref["out"]).max() <= TOL[L.dtype]
        ws[:64].fill_(0xAB)
        B_.moe_decode(*args)
        with pytest.raises(B_.OeaError) as err:
            B_.workspace_check(ws)
        assert err.value.code == B_.STATUS["OEA_ERR_WORKSPACE_STATE"]


def test_deterministic_combine_is_bit_reproducible(torch, B_, oracle):
    """oea_decode_ex.deterministic: the sum over a token's experts (Eq. 1) is taken in slot order, so
    `out` is the same bits on every call, on every kernel path; it still matches the oracle."""
    L30 = W.make_layer("qwen3_30b", 97, B=160)
    dev30 = {f: B_.to_device(getattr(L30, f)) for f in ("w_router", "w_gate", "w_up", "w_down")}
    cases = []
    for B in (16, 5, 64, 160):  # single kernel (two batch ranges), then router kernel + stage kernels
        Ls = W.Layer(**{**L30.__dict__, "B": B, "x": np.ascontiguousarray(L30.x[:B])})
        cases.append(("30b-shape B=%d" % B, Ls, dict(dev30, x=B_.to_device(Ls.x)), None, 3))
    Lm = W.make_layer("mid_bf16", 98)
    devm = {f: B_.to_device(getattr(Lm, f)) for f in ("x", "w_router", "w_gate", "w_up", "w_down")}
    Lf = W.make_layer("mid_f32", 99)
    devf = {f: B_.to_device(getattr(Lf, f)) for f in ("x", "w_router", "w_gate", "w_up", "w_down")}
    cases += [("mid_bf16 streaming kernels", Lm, devm, 2, 3), ("mid_bf16 generic kernels", Lm, devm, 1, 3),
              ("mid_f32", Lf, devf, None, 2)]
    for name, L, dev, path, k0 in cases:
        ws = B_.new_workspace(L.B, L.d, L.N, L.I, L.k, deterministic=True)
        first = None
        for it in range(20 if L.B <= 16 else 6):
            out, tap = B_.moe_decode(dev["x"], dev["w_router"], dev["w_gate"], dev["w_up"], dev["w_down"], L.k, k0, ws,
                                     taps=True, deterministic=True, kernel_path=path)
            torch.cuda.synchronize()
            o = out.cpu().numpy()
            if first is None:
                first = o
                err, ref = check_layer(oracle, L, k0, o, {n: v.cpu().numpy() for n, v in tap.items()}, "deterministic " + name)
                say("deterministic %s: T=%d err=%.2e" % (name, ref["n_active"], err))
            else:
                assert np.array_equal(o.view(np.uint32), first.view(np.uint32)), "%s: call %d differs" % (name, it)
        B_.workspace_check(ws)
    # the smaller workspace is refused when the flag is set
    L, dev = cases[0][1], cases[0][2]
    with pytest.raises(B_.OeaError) as e:
        B_.moe_decode(dev["x"], dev["w_router"], dev["w_gate"], dev["w_up"], dev["w_down"], L.k, 3,
                      B_.new_workspace(L.B, L.d, L.N, L.I, L.k), deterministic=True)
    assert e.value.code == B_.STATUS["OEA_ERR_WORKSPACE"]
    # padded tokens come out as zero rows
    mask = np.ones(L.B, np.uint8)
    mask[[2, 9]] = 0
    ws = B_.new_workspace(L.B, L.d, L.N, L.I, L.k, deterministic=True)
    out = B_.moe_decode(dev["x"], dev["w_router"], dev["w_gate"], dev["w_up"], dev["w_down"], L.k, 3, ws,
                        token_mask=torch.from_numpy(mask).cuda(), deterministic=True).cpu().numpy()
    assert (out[[2, 9]] == 0).all() and np.abs(out[0]).max() > 0


@pytest.mark.parametrize("d,N,B", [(128, 8, 80), (256, 8, 80), (256, 16, 80), (1024, 20, 40)], ids=lambda v: str(v))
def test_deterministic_bits_do_not_depend_on_the_result_buffer(torch, B_, d, N, B):
    """A workgroup with few results collects their gate and up sums in LDS, with more the results themselves, and with
    many it writes them as they come: all three add in one order.  With every expert selected (k0 = k = N) a
    token's row depends on that token alone, so its bits are the same alone (sums collected) and in a batch whose
    workgroups have more than 4096 results (8 experts x 2048 hidden units / 256 workgroups = 64 rows x 80 pairs;
    160 rows x about 30 pairs staged at once) or more than 8192 (128 rows x 80 pairs).  Rows of 8, 16 and 32
    lanes, fp32 hidden vectors."""
    I = 2048
    gen = torch.Generator(device="cuda")
    gen.manual_seed(d)
    x = torch.empty((B, d), device="cuda").normal_(generator=gen)
    w = [torch.empty(s, device="cuda").normal_(0.0, std, generator=gen)
         for s, std in (((N, d), d ** -0.5), ((N, I, d), 0.02), ((N, I, d), 0.02), ((N, d, I), 0.02))]

    def layer(rows):
        ws = B_.new_workspace(rows.shape[0], d, N, I, N, deterministic=True)
        return B_.moe_decode(rows.contiguous(), *w, N, N, ws, deterministic=True, kernel_path=3)

    dev = dict(zip(("x", "w_router", "w_gate", "w_up", "w_down"), [x] + w))
    ws = B_.new_workspace(B, d, N, I, N, deterministic=True)
    assert expert_kernels(torch, B_, dev, N, N, ws, 3, True) == [3, 3]
    whole = layer(x)
    for t in range(0, B, 16):
        assert torch.equal(layer(x[t:t + 1])[0], whole[t]), "token %d" % t


@pytest.mark.parametrize("B,crowded", [(32, (3, 77)), (128, ())], ids=["B32-crowded", "B128"])
def test_deterministic_bits_of_the_single_kernel(torch, B_, B, crowded):
    """The single-kernel layers with workgroups on both sides of the limit up to which both sums of a result are
    collected in LDS (B=32: two experts that every token selects are above it; B=128: experts with 11 pairs and
    more).  The same bits on every call, also while the shares of the workgroups still move with their measured
    speeds, and for every token the bits it has alone (k0 = k, so its weights do not depend on the batch)."""
    L, dev = big_layer(B_, "qwen3_30b", 2000)
    k = 8
    gen = torch.Generator(device="cuda")
    gen.manual_seed(B)
    x = torch.empty((B, L.d), device="cuda").normal_(generator=gen).bfloat16()
    bias = torch.zeros(L.N, device="cuda")
    bias[list(crowded)] = 20.0
    w = [dev[f] for f in ("w_router", "w_gate", "w_up", "w_down")]

    def layer(rows, ws):
        return B_.moe_decode(rows.contiguous(), *w, k, k, ws, router_bias=bias, deterministic=True, taps=True)

    ws = B_.new_workspace(B, L.d, L.N, L.I, k, deterministic=True)
    first, tap = layer(x, ws)
    first = first.clone()
    assert all(int((tap["expert_idx"] == e).sum()) == B for e in crowded)
    for it in range(60):
        assert torch.equal(layer(x, ws)[0], first), "call %d differs" % it
    ws1 = B_.new_workspace(1, L.d, L.N, L.I, k, deterministic=True)
    for t in range(B):
        out, tap1 = layer(x[t:t + 1], ws1)
        assert torch.equal(tap1["gate_w"][0], tap["gate_w"][t])
        assert torch.equal(out[0], first[t]), "token %d" % t
    B_.workspace_check(ws)


@pytest.mark.parametrize("case", [
    # three-kernel layers up to B = 128 (dot-product kernels, on both sides of the batches and pairs at which layers with
    # the atomic combine change their routing and expert kernels) ...
    (512, 64, 192, 8, "bf16", (16, 40, 96, 97), 128), (4096, 128, 192, 8, "bf16", (16, 64, 100), 128),
    (64, 16, 64, 4, "bf16", (20, 96), 120), (448, 24, 160, 8, "f32", (16, 90, 110), 128),
    # the single kernel, and at d=4096 the batches whose vectors do not fit its LDS (18 to 32 tokens)
    (2048, 128, 768, 8, "bf16", (5, 16, 33, 97), 128), (4096, 128, 1536, 8, "bf16", (9, 17, 24, 33), 100),
    # ... and layers above it (matrix cores)
    (1088, 64, 320, 6, "bf16", (130, 257), 400), (2048, 128, 768, 8, "bf16", (130, 200), 520),
    (4096, 128, 1536, 8, "bf16", (129, 400), 600)], ids=lambda c: "d%d-N%d-I%d-k%d-%s-B%d" % (c[:5] + c[6:]))
def test_deterministic_bits_do_not_depend_on_the_batch(torch, B_, case):
    """oea_decode_ex.deterministic on either side of B = 128: a token's row has the same bits whatever other tokens share
    the batch, in a batch of few active experts, with others that activate all, or beside padding (k0 = k, so its
    weights do not depend on the others either)."""
    d, N, I, k, dtype, sizes, B = case
    st = torch.bfloat16 if dtype == "bf16" else torch.float32
    gen = torch.Generator(device="cuda")
    gen.manual_seed(d + N)
    x = torch.empty((B, d), device="cuda").normal_(generator=gen).to(st)
    x[:sizes[0]] = x[torch.arange(sizes[0], device="cuda") % 2]  # two distinct tokens: at most 2 k active experts
    w = [torch.empty(s, device="cuda").normal_(0.0, std, generator=gen).to(st)
         for s, std in (((N, d), d ** -0.5), ((N, I, d), 0.02), ((N, I, d), 0.02), ((N, d, I), 0.02))]

    def layer(rows, mask=None):
        ws = B_.new_workspace(rows.shape[0], d, N, I, k, deterministic=True)
        out, tap = B_.moe_decode(rows.contiguous(), *w, k, k, ws, deterministic=True, taps=True, token_mask=mask)
        return out, tap["gate_w"], int(tap["n_active"][0])

    whole, weights, active = layer(x)
    seen = set()
    for n in sizes:
        out, gw, T = layer(x[:n])
        seen.add(T)
        assert torch.equal(gw, weights[:n]), "weights of %d tokens" % n
        assert torch.equal(out, whole[:n]), "rows of %d tokens" % n
    mask = torch.zeros(B, dtype=torch.uint8, device="cuda")
    mask[:sizes[0]] = 1
    out, gw, T = layer(x, mask)
    assert T <= 2 * k and (T < active or active == N <= 2 * k)
    assert torch.equal(gw[:sizes[0]], weights[:sizes[0]]) and torch.equal(out[:sizes[0]], whole[:sizes[0]])
    assert min(seen) == T


def test_cooperative_launch_option(torch, B_, oracle):
    """oea_decode_ex.cooperative: the single kernel through a cooperative launch (co-residency is then
    the runtime's guarantee); same results."""
    L = W.make_layer("qwen3_30b", 96, B=6)
    dev = {f: B_.to_device(getattr(L, f)) for f in ("x", "w_router", "w_gate", "w_up", "w_down")}
    ws = B_.new_workspace(L.B, L.d, L.N, L.I, L.k)
    for k0 in (2, 8):
        out, tap = B_.moe_decode(dev["x"], dev["w_router"], dev["w_gate"], dev["w_up"], dev["w_down"], L.k, k0, ws,
                                 taps=True, cooperative=True)
        torch.cuda.synchronize()
        check_layer(oracle, L, k0, out.cpu().numpy(), {n: v.cpu().numpy() for n, v in tap.items()},
                    "cooperative k0=%d" % k0)
    B_.workspace_check(ws)


def test_read_probe_runs_and_leaves_memory_alone(torch, B_):
    # the measurement aid only reads: the buffer is unchanged afterwards and the launch succeeds
    # for sizes that are not a multiple of its batch
    buf = torch.arange((3 << 20) + 4096, dtype=torch.int32, device="cuda:0")
    keep = buf.clone()
    B_.read_probe(buf)
    torch.cuda.synchronize()
    assert torch.equal(buf, keep)


def test_bounded_waits_report_a_timeout(torch, B_, oracle):
    """The single-kernel layer never waits forever: with the poll limit forced down to one poll its
    waits give up at once, every kernel still ends normally, and the workspace says so afterwards."""
    L = W.make_layer("qwen3_30b", 93, B=4)
    dev = {f: B_.to_device(getattr(L, f)) for f in ("x", "w_router", "w_gate", "w_up", "w_down")}
    ws = B_.new_workspace(L.B, L.d, L.N, L.I, L.k)
    args = (dev["x"], dev["w_router"], dev["w_gate"], dev["w_up"], dev["w_down"], L.k, 2, ws)
    good = B_.moe_decode(*args).cpu().numpy()
    B_.workspace_check(ws)  # nothing gave up
    say("forcing the waits of one call to give up (poll limit 1)")
    B_.moe_decode(*args, spin_limit=1)
    with pytest.raises(B_.OeaError) as err:
        B_.workspace_check(ws)
    assert err.value.code == -8
    # the record is sticky until the workspace is prepared again; then the layer is right again
    B_.workspace_init(ws)
    again = B_.moe_decode(*args).cpu().numpy()
    B_.workspace_check(ws)
    ref = oracle.moe_decode(L.x, L.w_router, L.w_gate, L.w_up, L.w_down, L.k, 2)
    for got in (good, again):
        assert np.abs(got - ref["out"]).max() / np.abs(ref["out"]).max() <= TOL[L.dtype]


@pytest.mark.parametrize("shape", [
    # rows that are no multiple of a workgroup's eight granules, inner dimensions of one, three and five slabs, a granule
    # count without a divisor below nine; one pair per expert; more tokens on an expert than a pass holds
    (130, 64, 24, 64, 4, 2, False), (129, 192, 40, 320, 3, 1, False), (200, 576, 6, 176 * 4, 2, 2, True),
    (150, 320, 512, 192, 1, 1, False), (640, 128, 3, 64, 2, 1, True)],
    ids=lambda c: "B%d-d%d-N%d-I%d-k%d-k0%d%s" % (c[:6] + ("-det" if c[6] else "",)))
def test_matrix_core_granules(torch, B_, oracle, shape):
    """The matrix-core stages where a job has fewer granules or slabs than the ring and the wavefronts could take."""
    B, d, N, I, k, k0, det = shape
    L = W.make_layer("toy", 1700 + B, d=d, I=I, N=N, B=B, k=k, dtype="bf16")
    mask = np.ones(B, np.uint8)
    mask[B // 2] = 0
    ws = B_.new_workspace(B, d, N, I, k, deterministic=det)
    dev = {f: B_.to_device(getattr(L, f)) for f in ("x", "w_router", "w_gate", "w_up", "w_down")}
    assert expert_kernels(torch, B_, dev, k, k0, ws, 4, det) == [4, 4]
    outs = []
    for _ in range(2):
        out, tap = B_.moe_decode(dev["x"], dev["w_router"], dev["w_gate"], dev["w_up"], dev["w_down"], k, k0, ws, taps=True,
                                 token_mask=torch.from_numpy(mask).cuda(), deterministic=det, kernel_path=4)
        torch.cuda.synchronize()
        outs.append(out.cpu().numpy())
        check_layer(oracle, L, k0, outs[-1], {n: v.cpu().numpy() for n, v in tap.items()}, str(shape), mask=mask)
    if det:
        assert np.array_equal(outs[0].view(np.uint32), outs[1].view(np.uint32))


@pytest.mark.parametrize("det", [False, True], ids=["atomics", "det"])
@pytest.mark.parametrize("shape", [
    # I in whole granules of the gate/up stage and no whole slabs of the down stage, and d the other way round (whole granules of
    # the down stage, no whole slabs of the gate/up stage); automatic choice above B = 128 and below
    (40, 512, 6, 80, 3, 2, 4, [4, None]), (200, 512, 6, 80, 3, 2, None, [4, None]), (100, 512, 6, 80, 3, 2, None, [None, None]),
    (200, 1024, 24, 1040, 4, 2, None, [4, None]), (40, 96, 6, 64, 3, 2, 4, [None, 4]), (200, 96, 6, 128, 3, 2, None, [None, 4])],
    ids=lambda c: "B%d-d%d-N%d-I%d-k%d-k0%d-path%s" % c[:7])
def test_one_stage_on_the_matrix_cores(torch, B_, oracle, shape, det):
    """Layers of which only one stage fits the matrix-core kernel: the other one keeps the dot products, and they hand the
    hidden vectors over."""
    B, d, N, I, k, k0, path, stages = shape
    L = W.make_layer("toy", 3300 + B, d=d, I=I, N=N, B=B, k=k, dtype="bf16")
    ws = B_.new_workspace(B, d, N, I, k, deterministic=det)
    dev = {f: B_.to_device(getattr(L, f)) for f in ("x", "w_router", "w_gate", "w_up", "w_down")}
    got = expert_kernels(torch, B_, dev, k, k0, ws, path, det)
    assert all(g == 4 if s == 4 else g in (1, 3) for g, s in zip(got, stages)), got
    out, tap = B_.moe_decode(dev["x"], dev["w_router"], dev["w_gate"], dev["w_up"], dev["w_down"], k, k0, ws, taps=True,
                             deterministic=det, kernel_path=path)
    torch.cuda.synchronize()
    check_layer(oracle, L, k0, out.cpu().numpy(), {n: v.cpu().numpy() for n, v in tap.items()}, str(shape))


@pytest.mark.parametrize("det", [False, True], ids=["atomics", "det"])
@pytest.mark.parametrize("shape", [
    # one, two and three slabs of the down stage's inner dimension, with 4 to 40 of its granules per workgroup (jobs of
    # up to eight, of different experts); few pairs per expert, full groups of 16 and a rest, several passes
    (16, 2048, 128, 64, 8, 3), (200, 2048, 160, 64, 8, 8), (300, 2048, 96, 128, 6, 2), (130, 4096, 64, 192, 8, 3),
    (700, 8192, 4, 64, 2, 2)],
    ids=lambda c: "B%d-d%d-N%d-I%d-k%d-k0%d" % c)
def test_matrix_core_results_of_consecutive_jobs(torch, B_, oracle, shape, det):
    """The down stage where a workgroup walks several jobs of several wavefronts each, of different experts or passes, one
    to three slabs apart: every job's results carry the tokens and gate weights of its own pairs."""
    B, d, N, I, k, k0 = shape
    L = W.make_layer("toy", 2900 + B, d=d, I=I, N=N, B=B, k=k, dtype="bf16")
    ws = B_.new_workspace(B, d, N, I, k, deterministic=det)
    dev = {f: B_.to_device(getattr(L, f)) for f in ("x", "w_router", "w_gate", "w_up", "w_down")}
    assert expert_kernels(torch, B_, dev, k, k0, ws, 4, det) == [4, 4]
    for call in range(3):
        out, tap = B_.moe_decode(dev["x"], dev["w_router"], dev["w_gate"], dev["w_up"], dev["w_down"], k, k0, ws, taps=True,
                                 deterministic=det, kernel_path=4)
        torch.cuda.synchronize()
        out = out.cpu().numpy()
        if call == 0:
            first = out
            check_layer(oracle, L, k0, out, {n: v.cpu().numpy() for n, v in tap.items()}, str(shape))
        elif det:
            assert np.array_equal(out.view(np.uint32), first.view(np.uint32)), "call %d differs" % call
        else:  # fp32 sums of k products in another order
            assert np.abs(out - first).max() <= 2e-6 * k * np.abs(first).max(), "call %d" % call
