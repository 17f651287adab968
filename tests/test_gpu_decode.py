"""GPU parity of the fused decode against the FP64 oracle.

Gates: BC1 texel decode bit-exact; outputs within 1e-5 relative (FP32),
2e-3 absolute (FP16) and 3e-2 absolute (FP8 E4M3) of the exact FP64 result.
Full-size workloads (4096^2 pixels) are checked on every pixel against the
oracle's decode of the whole image (a few seconds on the host's cores), in
the benchmark's 8x8-tile pixel order and in row-major order; small workloads
on every pixel too.
"""
import numpy as np
import pytest
import torch

import ntc_inputs as I
import oracle as O

pytestmark = pytest.mark.gpu

TOL_F32_REL = 1e-5
TOL_F16_ABS = 2e-3
TOL_FP8_ABS = 3e-2
# BF16 keeps 8 significant bits against FP16's 11: unit roundoff 2^-8 is
# 8x that of FP16, so its gate is 8x the FP16 one
TOL_BF16_ABS = 8 * TOL_F16_ABS


def _ntc():
    import paper_2506_06040_amd as ntc
    return ntc


def _report(name, got, ref):
    err = np.abs(got.astype(np.float64) - ref)
    mx = err.max(axis=0)
    rms = np.sqrt((err ** 2).mean(axis=0))
    print(f"\n[{name}] n={got.shape[0]} per-channel max {np.array2string(mx, precision=2)} "
          f"rms {np.array2string(rms, precision=2)}", flush=True)
    return err


def _gpu_case(lat_np, Ws, bs, shift, address="clamp"):
    ntc = _ntc()
    lat = ntc.Latents(lat_np, shift=shift, address=address)
    mlp = ntc.Mlp(Ws, bs)
    return lat, mlp


def _oracle_case(lat_np, Ws, bs, shift, address="clamp"):
    return O.Latents(lat_np, shift=shift, address=O.CLAMP if address == "clamp" else O.WRAP), O.Mlp(Ws, bs)


def _sample_index(n, k, seed):
    rng = np.random.default_rng(seed)
    idx = np.concatenate([np.arange(min(n, 256)), np.arange(max(0, n - 256), n), rng.integers(0, n, k)])
    return np.unique(idx)


# ---------------------------------------------------------------------------
def test_bc1_texels_bitexact():
    ntc = _ntc()
    for wl in (I.WORKLOADS["c1"], I.WORKLOADS["c2"]):
        print(f"[texels] {wl.name}", flush=True)
        lat_np = I.bc1_pyramid(I.streams(wl.seed)[0], wl.latent_sizes)
        lat = ntc.Latents(lat_np)
        for k in range(len(lat_np)):
            val, num = ntc.bc1_decode_texels(lat, k)
            val = val.cpu().numpy()
            num = num.cpu().numpy().astype(np.int64)
            onum, oden, oval = O.bc1_level(lat_np[k])
            den6 = np.array([186, 378, 186], np.int64)
            # num / den6 == onum / oden exactly
            assert np.array_equal(num * oden.astype(np.int64), onum.astype(np.int64) * den6), (wl.name, k)
            assert np.array_equal(val, oval.astype(np.float32)), (wl.name, k)


def test_plain_f32_c1_all_pixels():
    ntc = _ntc()
    wl = I.WORKLOADS["c1"]
    lat_np, Ws, bs, uv = I.make_workload(wl)
    lat, mlp = _gpu_case(lat_np, Ws, bs, wl.shift)
    out = ntc.decode(lat, mlp, torch.from_numpy(uv).cuda(), compute="f32").cpu().numpy()
    olat, omlp = _oracle_case(lat_np, Ws, bs, wl.shift)
    ref = O.decode(olat, omlp, uv)
    err = _report("c1 f32", out, ref)
    assert np.all(err <= TOL_F32_REL * np.abs(ref))


@pytest.mark.parametrize("compute,tol", [("f16", TOL_F16_ABS), ("bf16", TOL_BF16_ABS), ("f32", None),
                                         ("fp8", TOL_FP8_ABS)])
def test_c1_shape_variants(compute, tol):
    """Random biases, ragged sizes, wrap addressing, no shift, uv outside [0,1],
    fewer levels, 9 output channels."""
    ntc = _ntc()
    rng = np.random.default_rng(21)
    cases = [
        dict(n=1000, levels=4, address="clamp", shift=I.PAPER_SHIFT, dims=(14, 32, 32, 8), uvr=(0, 1)),
        dict(n=777, levels=4, address="wrap", shift=I.PAPER_SHIFT, dims=(14, 32, 32, 8), uvr=(-0.3, 1.4)),
        dict(n=65, levels=4, address="clamp", shift=I.NO_SHIFT, dims=(14, 64, 64, 64, 8), uvr=(-0.1, 1.1)),
        dict(n=1, levels=4, address="clamp", shift=I.PAPER_SHIFT, dims=(14, 16, 9), uvr=(0, 1)),
        dict(n=300, levels=2, address="clamp", shift=I.PAPER_SHIFT, dims=(8, 16, 16, 16, 16, 4), uvr=(0, 1)),
        dict(n=500, levels=3, address="clamp", shift=I.PAPER_SHIFT, dims=(11, 32, 9), uvr=(0, 1)),
        dict(n=129, levels=4, address="clamp", shift=I.PAPER_SHIFT, dims=(14, 64, 16), uvr=(0, 1)),
    ]
    for ci, c in enumerate(cases):
        sizes = [(64, 32), (32, 32), (16, 8), (8, 8)][:c["levels"]]
        lat_np = I.bc1_pyramid(rng, sizes)
        Ws, bs = I.xavier_mlp(rng, c["dims"], bias="normal")
        uv = (rng.random((c["n"], 2)) * (c["uvr"][1] - c["uvr"][0]) + c["uvr"][0]).astype(np.float32)
        lat, mlp = _gpu_case(lat_np, Ws, bs, c["shift"], c["address"])
        packed = None
        if compute == "fp8":
            # ranges calibrated on the decoded coordinates themselves
            packed = ntc.pack(mlp, "fp8", act_amax=ntc.calibrate_fp8(lat, mlp, torch.from_numpy(uv).cuda()))
        out = ntc.decode(lat, mlp, torch.from_numpy(uv).cuda(), compute=compute, packed=packed).cpu().numpy()
        olat, omlp = _oracle_case(lat_np, Ws, bs, c["shift"], c["address"])
        ref = O.decode(olat, omlp, uv)
        err = _report(f"variant {ci} {compute}", out, ref)
        if compute == "f32":
            assert np.all(err <= TOL_F32_REL * np.abs(ref)), ci
        else:
            assert np.all(err <= tol), ci


def test_f16_c1_all_pixels_and_emulation():
    ntc = _ntc()
    wl = I.WORKLOADS["c1"]
    lat_np, Ws, bs, uv = I.make_workload(wl, bias="normal")
    lat, mlp = _gpu_case(lat_np, Ws, bs, wl.shift)
    out = ntc.decode(lat, mlp, torch.from_numpy(uv).cuda(), compute="f16").cpu().numpy()
    olat, omlp = _oracle_case(lat_np, Ws, bs, wl.shift)
    ref = O.decode(olat, omlp, uv)
    err = _report("c1 f16", out, ref)
    assert np.all(err <= TOL_F16_ABS)
    # diagnostic bound: the oracle with the same binary16 rounding of
    # inputs/weights/activations differs only by accumulation order and the
    # FP32 feature path
    emu = O.decode(olat, O.Mlp(Ws, bs, precision=O.FP16), uv)
    assert np.max(np.abs(out - emu)) <= 2e-4


def test_staged_equals_direct_and_deterministic():
    ntc = _ntc()
    wl = I.WORKLOADS["c1"]
    lat_np, Ws, bs, uv = I.make_workload(wl, bias="normal")
    lat, mlp = _gpu_case(lat_np, Ws, bs, wl.shift)
    uvt = torch.from_numpy(uv).cuda()
    for compute in ("f16", "bf16"):
        packed = ntc.pack(mlp, compute)
        a = ntc.decode(lat, mlp, uvt, compute=compute, packed=packed)
        b = ntc.decode(lat, mlp, uvt, compute=compute, packed=packed)
        c = ntc.decode(lat, mlp, uvt, compute=compute, packed=packed, cfg=ntc.tile_cfg(stage_capacity=64))
        d = ntc.decode(lat, mlp, uvt, compute=compute, packed=packed, cfg=ntc.tile_cfg(waves_per_cu=3))
        e = ntc.decode(lat, mlp, uvt, compute=compute, packed=packed, cfg=ntc.tile_cfg(waves_per_cu=1))
        f = ntc.decode(lat, mlp, uvt[:4099], compute=compute, packed=packed, cfg=ntc.tile_cfg(tiles_per_iter=8))
        torch.cuda.synchronize()
        assert torch.equal(a, b)
        assert torch.equal(a, c)
        assert torch.equal(a, d)
        assert torch.equal(a, e)
        assert torch.equal(a[:4099], f)


def _white_pyramid(sizes):
    """BC1 levels whose every texel is (1, 1, 1): both endpoints 0xFFFF."""
    return [np.full((h // 4, w // 4), 0xFFFFFFFF, np.uint64) for (w, h) in sizes]


def test_f16_unit_relu_at_its_bound():
    """FP16 images scale hidden neuron i of layer l by 2^-e(l, i) so that ReLU
    is the conversion's [0, 1] clamp. Here layer 1 reaches its interval bound:
    positive weights, white latents and u = v = 1 make every input 1, and
    each row sums to just below a power of two, so a scale one binade too
    small would saturate. Parity with the oracle, and the staged path (clamp)
    equals the direct path (max) bit for bit."""
    ntc = _ntc()
    rng = np.random.default_rng(31)
    sizes = [(64, 64), (32, 32), (16, 16), (8, 8)]
    lat_np = _white_pyramid(sizes)
    W1 = rng.random((64, 14))
    W1 /= W1.sum(1, keepdims=True)
    c = rng.uniform(1.5, 1.98, 64) * 2.0 ** rng.integers(-2, 3, 64)
    Ws = [(W1 * (0.9 * c)[:, None]).astype(np.float32), (rng.random((64, 64)) * 0.05).astype(np.float32),
          (rng.random((64, 64)) * 0.05).astype(np.float32), I.xavier_mlp(rng, (64, 8))[0][0]]
    bs = [(0.1 * c).astype(np.float32), np.full(64, 0.01, np.float32), np.full(64, 0.01, np.float32),
          np.zeros(8, np.float32)]
    n = 4096
    uv = (1.0 - rng.random((n, 2)) / 8).astype(np.float32)
    uv[::7] = 1.0
    lat, mlp = _gpu_case(lat_np, Ws, bs, I.PAPER_SHIFT)
    uvt = torch.from_numpy(uv).cuda()
    packed = ntc.pack(mlp, "f16")
    out = ntc.decode(lat, mlp, uvt, compute="f16", packed=packed)
    # 64 texels of staging cannot hold these footprints: every span direct
    direct = ntc.decode(lat, mlp, uvt, compute="f16", packed=packed, cfg=ntc.tile_cfg(stage_capacity=64))
    olat, omlp = _oracle_case(lat_np, Ws, bs, I.PAPER_SHIFT)
    ref = O.decode(olat, omlp, uv)
    err = _report("unit relu at bound", out.cpu().numpy(), ref)
    assert np.all(err <= TOL_F16_ABS)
    assert torch.equal(out, direct)


def test_f16_large_bounds_parity():
    """A neuron whose interval bound exceeds 2^10 (bias 3000 on one layer-2
    neuron, whose outgoing weights are zero) leaves the FP16 image unscaled,
    with max-based ReLU everywhere: parity with the oracle, and the staged and
    direct paths agree bit for bit."""
    ntc = _ntc()
    rng = np.random.default_rng(32)
    lat_np = I.bc1_pyramid(rng, [(64, 64), (32, 32), (16, 16), (8, 8)])
    Ws, bs = I.xavier_mlp(rng, (14, 64, 64, 64, 8), bias="normal")
    bs[1][5] = 3000.0
    Ws[2][:, 5] = 0.0
    uv = I.pixel_uv(64, 48)
    lat, mlp = _gpu_case(lat_np, Ws, bs, I.PAPER_SHIFT)
    uvt = torch.from_numpy(uv).cuda()
    packed = ntc.pack(mlp, "f16")
    out = ntc.decode(lat, mlp, uvt, compute="f16", packed=packed)
    direct = ntc.decode(lat, mlp, uvt, compute="f16", packed=packed, cfg=ntc.tile_cfg(stage_capacity=64))
    olat, omlp = _oracle_case(lat_np, Ws, bs, I.PAPER_SHIFT)
    ref = O.decode(olat, omlp, uv)
    err = _report("large bounds f16", out.cpu().numpy(), ref)
    assert np.all(err <= TOL_F16_ABS)
    assert torch.equal(out, direct)


def test_f16_scaled_output_weights_stay_finite():
    """A hidden neuron whose bound needs the largest scale (bias 700: 2^-10)
    and whose outgoing weights are 100: scaled, those weights would be
    102400, beyond FP16's finite range, and the neuron's zero outputs would
    turn the outputs into NaN (0 * inf). The packer leaves such an image
    unscaled: parity with the oracle on every pixel, no NaN.

    The neuron reads level 0's red channel only (weight -1400): the level is
    red (1) on its left half and black (0) on its right half and the samples
    sit on its texel centres, so the neuron is 700 (on) or -700 (off) exactly
    and its large output weights never meet a small activation."""
    ntc = _ntc()
    rng = np.random.default_rng(34)
    red = np.uint64(0xF800 | (0xF800 << 16))
    lvl0 = np.zeros((16, 16), np.uint64)
    lvl0[:, :8] = red
    lat_np = [lvl0] + I.bc1_pyramid(rng, [(32, 32), (16, 16), (8, 8)])
    Ws, bs = I.xavier_mlp(rng, (14, 32, 8), bias="normal")
    Ws[0][0, :] = 0.0
    Ws[0][0, 0] = -1400.0
    bs[0][0] = 700.0
    Ws[1][:, 0] = 0.001
    Ws[1][3, 0] = 100.0
    shift = ((0.0, 0.0), (0.5, 0.5), (0.0, 0.0), (0.5, 0.5))
    uv = I.pixel_uv(64, 64, order="tiled")
    lat, mlp = _gpu_case(lat_np, Ws, bs, shift)
    uvt = torch.from_numpy(uv).cuda()
    olat, omlp = _oracle_case(lat_np, Ws, bs, shift)
    ref = O.decode(olat, omlp, uv)
    x0 = O.features(olat, uv)[:, 0]
    assert set(np.unique(x0)) == {0.0, 1.0}
    for cfg in (None, ntc.tile_cfg(stage_capacity=64)):
        out = ntc.decode(lat, mlp, uvt, compute="f16", cfg=cfg)
        assert torch.isfinite(out).all()
        err = _report("f16 large output weights", out.cpu().numpy(), ref)
        assert np.all(err <= TOL_F16_ABS)


def test_non_finite_and_far_uv():
    """uv outside the unit square: NaN, +-inf and huge finite values. The
    sampling position is limited before the taps are formed (NaN to the left
    or top edge, everything else clamped to the edge texels), so no access
    leaves a level; u and v themselves are features, so the outputs of
    non-finite samples are not specified. Finite samples of the same launch
    equal a launch without the others bit for bit on every path (FP32, FP16,
    E4M3; staged and direct); huge finite coordinates with zero weights on
    the u, v features decode to the edge texels (FP32 path, against the
    oracle)."""
    ntc = _ntc()
    rng = np.random.default_rng(36)
    lat_np = I.bc1_pyramid(rng, [(64, 64), (32, 32), (16, 16), (8, 8)])
    Ws, bs = I.xavier_mlp(rng, (14, 32, 32, 8), bias="normal")
    Ws[0][:, 12:] = 0.0
    lat, mlp = _gpu_case(lat_np, Ws, bs, I.PAPER_SHIFT)
    clean = rng.random((1000, 2)).astype(np.float32)
    bad = np.array([[np.nan, 0.5], [0.5, np.nan], [np.inf, 0.2], [-np.inf, 0.7], [0.3, np.inf],
                    [0.6, -np.inf], [np.nan, np.nan], [np.inf, -np.inf]], np.float32)
    far = np.array([[1e10, 0.5], [-1e10, 0.25], [0.5, 3e38], [0.75, -3e38], [-3e38, 3e38], [2.5, -1.5]],
                   np.float32)
    mixed = np.concatenate([clean[:300], bad, clean[300:600], far, clean[600:]])
    is_clean = np.ones(mixed.shape[0], bool)
    is_clean[300:300 + len(bad)] = False
    is_clean[600 + len(bad):600 + len(bad) + len(far)] = False
    cal = torch.from_numpy(I.calibration_uv(4096)).cuda()
    p8 = ntc.pack(mlp, "fp8", act_amax=ntc.calibrate_fp8(lat, mlp, cal))
    for compute, packed in (("f32", None), ("f16", None), ("fp8", p8)):
        for cfg in (None, ntc.tile_cfg(stage_capacity=64)):
            if compute == "f32" and cfg is not None:
                continue
            a = ntc.decode(lat, mlp, torch.from_numpy(mixed).cuda(), compute=compute, packed=packed, cfg=cfg)
            b = ntc.decode(lat, mlp, torch.from_numpy(clean).cuda(), compute=compute, packed=packed, cfg=cfg)
            torch.cuda.synchronize()
            assert torch.equal(a[torch.from_numpy(is_clean).cuda()], b), (compute, cfg is None)
    out = ntc.decode(lat, mlp, torch.from_numpy(far).cuda(), compute="f32").cpu().numpy()
    olat, omlp = _oracle_case(lat_np, Ws, bs, I.PAPER_SHIFT)
    # the oracle clamps each tap; the kernel limits the position first: the
    # same edge texels either way
    edge = np.clip(far.astype(np.float64), -4.0, 4.0)
    ref = O.decode(olat, omlp, edge)
    err = _report("far uv f32", out, ref)
    assert np.all(err <= TOL_F32_REL * np.abs(ref))


def test_random_uv_fallback_parity():
    """Random uv: tile footprints exceed the staging capacity -> direct fetches."""
    ntc = _ntc()
    wl = I.WORKLOADS["c2"]
    s_lat, s_mlp, _, _ = I.streams(wl.seed)
    lat_np = I.bc1_pyramid(s_lat, wl.latent_sizes)
    Ws, bs = I.xavier_mlp(s_mlp, wl.dims, bias="normal")
    uv = I.random_uv(np.random.default_rng(5), 20000)
    lat, mlp = _gpu_case(lat_np, Ws, bs, wl.shift)
    out = ntc.decode(lat, mlp, torch.from_numpy(uv).cuda(), compute="f16").cpu().numpy()
    olat, omlp = _oracle_case(lat_np, Ws, bs, wl.shift)
    ref = O.decode(olat, omlp, uv)
    err = _report("random uv f16", out, ref)
    assert np.all(err <= TOL_F16_ABS)


def test_empty_and_out_f16():
    ntc = _ntc()
    rng = np.random.default_rng(3)
    lat_np = I.bc1_pyramid(rng, [(32, 32), (16, 16), (8, 8), (4, 4)])
    Ws, bs = I.xavier_mlp(rng, (14, 32, 32, 8), bias="normal")
    lat, mlp = _gpu_case(lat_np, Ws, bs, I.PAPER_SHIFT)
    empty = ntc.decode(lat, mlp, torch.zeros((0, 2), device="cuda"), compute="f16")
    assert empty.shape == (0, 8)
    uv = rng.random((333, 2)).astype(np.float32)
    o16 = ntc.decode(lat, mlp, torch.from_numpy(uv).cuda(), compute="f16", out_dtype=torch.float16)
    o32 = ntc.decode(lat, mlp, torch.from_numpy(uv).cuda(), compute="f16", out_dtype=torch.float32)
    assert o16.dtype == torch.float16
    assert torch.equal(o16, o32.to(torch.float16))


# ---------------------------------------------------------------------------
# Full-size workloads (4096^2 pixels), every pixel
# ---------------------------------------------------------------------------
@pytest.fixture(scope="module")
def c2_case():
    wl = I.WORKLOADS["c2"]
    lat_np, Ws, bs, uv = I.make_workload(wl)
    ntc = _ntc()
    lat, mlp = _gpu_case(lat_np, Ws, bs, wl.shift)
    uvt = torch.from_numpy(uv).cuda()
    olat, omlp = _oracle_case(lat_np, Ws, bs, wl.shift)
    print(f"\n[c2] oracle over all {uv.shape[0]} pixels", flush=True)
    ref = O.decode(olat, omlp, uv)
    idx = _sample_index(uv.shape[0], 30000, 7)
    return dict(wl=wl, lat_np=lat_np, Ws=Ws, bs=bs, uv=uv, lat=lat, mlp=mlp, uvt=uvt, olat=olat, omlp=omlp,
                idx=idx, ref=ref)


def _check_all(name, out, ref, tol=None, rel=None):
    """Every pixel against the oracle (absolute gate `tol` or relative `rel`)."""
    assert torch.isfinite(out).all(), name
    err = _report(name, out.cpu().numpy(), ref)
    if tol is not None:
        assert np.all(err <= tol), name
    if rel is not None:
        assert np.all(err <= rel * np.abs(ref)), name
    return err


def test_c2_f16_full_size(c2_case):
    ntc = _ntc()
    c = c2_case
    out = ntc.decode(c["lat"], c["mlp"], c["uvt"], compute="f16")
    _check_all("c2 f16 4096^2 all pixels", out, c["ref"], tol=TOL_F16_ABS)


def test_c2_f16_rowmajor_full_size(c2_case):
    """The same 16.7 M samples in row-major pixel order (spans are 256-pixel
    runs of one row instead of four 8x8 tiles): every pixel against the
    oracle, and bit for bit the tiled launch's result for the same sample."""
    ntc = _ntc()
    c = c2_case
    perm = I.tiled_to_rowmajor(4096, 4096)
    uv_rm = np.empty_like(c["uv"])
    uv_rm[perm] = c["uv"]
    ref_rm = np.empty_like(c["ref"])
    ref_rm[perm] = c["ref"]
    out_rm = ntc.decode(c["lat"], c["mlp"], torch.from_numpy(uv_rm).cuda(), compute="f16")
    _check_all("c2 f16 4096^2 row-major all pixels", out_rm, ref_rm, tol=TOL_F16_ABS)
    out_t = ntc.decode(c["lat"], c["mlp"], c["uvt"], compute="f16")
    assert torch.equal(out_rm[torch.from_numpy(perm).cuda()], out_t)


def test_c2_bf16_full_size(c2_case):
    ntc = _ntc()
    c = c2_case
    out = ntc.decode(c["lat"], c["mlp"], c["uvt"], compute="bf16")
    _check_all("c2 bf16 4096^2 all pixels", out, c["ref"], tol=TOL_BF16_ABS)


def test_varA_layout_parity():
    """Variant A of the paper's latent layouts: levels at W, W, W/2, W/2 (the
    default workloads use variant B, W, W/2, W/4, W/8)."""
    ntc = _ntc()
    rng = np.random.default_rng(51)
    w = 256
    sizes = [(w, w), (w, w), (w // 2, w // 2), (w // 2, w // 2)]
    lat_np = I.bc1_pyramid(rng, sizes)
    Ws, bs = I.xavier_mlp(rng, (14, 64, 64, 64, 8), bias="normal")
    uv = I.pixel_uv(w, w, order="tiled")
    lat, mlp = _gpu_case(lat_np, Ws, bs, I.PAPER_SHIFT)
    uvt = torch.from_numpy(uv).cuda()
    olat, omlp = _oracle_case(lat_np, Ws, bs, I.PAPER_SHIFT)
    ref = O.decode(olat, omlp, uv)
    for compute, tol in (("f16", TOL_F16_ABS), ("bf16", TOL_BF16_ABS)):
        out = ntc.decode(lat, mlp, uvt, compute=compute)
        direct = ntc.decode(lat, mlp, uvt, compute=compute, cfg=ntc.tile_cfg(stage_capacity=64))
        err = _report(f"varA {compute}", out.cpu().numpy(), ref)
        assert np.all(err <= tol)
        assert torch.equal(out, direct)


def test_c2_f32_full_size(c2_case):
    ntc = _ntc()
    c = c2_case
    out = ntc.decode(c["lat"], c["mlp"], c["uvt"], compute="f32")
    _check_all("c2 f32 4096^2 all pixels", out, c["ref"], rel=TOL_F32_REL)


# E4M3 against the oracle's E4M3 emulation (precision FP8_F16: same scales,
# same roundings of weights and activations, hidden activations through
# binary16, exact accumulation). The two differ where an FP32
# accumulation lands on the other side of an E4M3 rounding midpoint than the
# exact sum: a pre-activation z evaluated by FP32 fused multiply-adds is off
# by at most about n u sum|terms| (n <= 64, u = 2^-24), i.e. within ~4e-6 of
# sum|terms|, while midpoints of E4M3 sit 2^-4 .. 2^-3 of the value apart, so
# with sum|terms| / |z| of order 10 a conversion flips with probability
# below 2 * 4e-6 * 10 / 2^-4 ~ 1.3e-3 and a pixel (206 conversions) rarely
# sees more than one. Pixels without a flip agree to FP32 rounding; a flip
# moves one activation by one E4M3 step, which the gate tolerates. Measured
# on the C4 workload: 98.9 % of sampled pixels within 1e-4, max 5.8e-3.
FP8_EMU_MATCH_TOL = 1e-4
FP8_EMU_MIN_MATCH = 0.95


def test_c4_fp8_full_size(c2_case):
    ntc = _ntc()
    c = c2_case
    cal = torch.from_numpy(I.calibration_uv()).cuda()
    amax = ntc.calibrate_fp8(c["lat"], c["mlp"], cal)
    # the calibration is checked against the oracle's own ranges
    oam = O.layer_amax(c["olat"], c["omlp"], I.calibration_uv())
    assert np.allclose(amax.cpu().numpy(), oam, rtol=1e-5)
    packed = ntc.pack(c["mlp"], "fp8", act_amax=amax)
    out = ntc.decode(c["lat"], c["mlp"], c["uvt"], compute="fp8", packed=packed)
    _check_all("c4 fp8 4096^2 all pixels", out, c["ref"], tol=TOL_FP8_ABS)
    got = out[torch.from_numpy(c["idx"]).cuda()].cpu().numpy()
    ws, as_ = O.fp8_scales(c["Ws"], oam, pow2=True)
    emu = O.decode_index(c["olat"], O.Mlp(c["Ws"], c["bs"], precision=O.FP8_F16, w_scale=ws, a_scale=as_), c["uv"],
                         c["idx"])
    d = np.abs(got - emu).max(axis=1)
    match = float(np.mean(d <= FP8_EMU_MATCH_TOL))
    print(f"[c4 fp8 vs emulation] max {d.max():.3g} rms {np.sqrt((d**2).mean()):.3g} "
          f"pixels within {FP8_EMU_MATCH_TOL:g}: {match:.4f}", flush=True)
    assert match >= FP8_EMU_MIN_MATCH
    assert d.max() <= TOL_FP8_ABS


def test_extra_output_row_keeps_other_channels_bit_identical():
    """Output rows are computed independently: a 9-output network whose first
    8 rows are those of an 8-output network reproduces those 8 channels bit
    for bit. The 9-channel rows leave through LDS-staged contiguous stores
    (complete 32-pixel tiles) and single stores (the ragged last tile), the
    8-channel rows through 16-byte stores per lane; staged and direct
    sampling. The ninth channel is checked against the oracle."""
    ntc = _ntc()
    rng = np.random.default_rng(53)
    sizes = [(256, 256), (128, 128), (64, 64), (32, 32)]
    lat_np = I.bc1_pyramid(rng, sizes)
    Ws, bs = I.xavier_mlp(rng, (14, 64, 64, 64, 8), bias="normal")
    row = (rng.standard_normal((1, 64)) * 0.15).astype(np.float32)
    W9 = list(Ws[:-1]) + [np.concatenate([Ws[-1], row], 0)]
    b9 = list(bs[:-1]) + [np.concatenate([bs[-1], np.float32([0.25])])]
    uv = I.pixel_uv(512, 128, order="tiled")[:512 * 128 - 37]
    lat, mlp8 = _gpu_case(lat_np, Ws, bs, I.PAPER_SHIFT)
    _, mlp9 = _gpu_case(lat_np, W9, b9, I.PAPER_SHIFT)
    uvt = torch.from_numpy(uv).cuda()
    olat, omlp9 = _oracle_case(lat_np, W9, b9, I.PAPER_SHIFT)
    ref9 = O.decode(olat, omlp9, uv)[:, 8:9]
    for compute, tol in (("f16", TOL_F16_ABS), ("bf16", TOL_BF16_ABS)):
        for cfg in (None, ntc.tile_cfg(stage_capacity=64)):
            o8 = ntc.decode(lat, mlp8, uvt, compute=compute, cfg=cfg)
            o9 = ntc.decode(lat, mlp9, uvt, compute=compute, cfg=cfg)
            assert torch.equal(o9[:, :8], o8), (compute, cfg is None)
            err = _report(f"9th channel {compute}", o9[:, 8:9].cpu().numpy(), ref9)
            assert np.all(err <= tol)


@pytest.mark.parametrize("compute,tol", [("f16", TOL_F16_ABS), ("bf16", TOL_BF16_ABS), ("fp8", TOL_FP8_ABS)])
def test_span_boundaries(compute, tol):
    """Pixel counts around the 256- and 512-pixel spans (the span length
    depends on the network shape) on coherent uv, so that the spans are
    staged: every pixel against the oracle, nothing written past the end."""
    ntc = _ntc()
    rng = np.random.default_rng(31)
    sizes = [(64, 64), (32, 32), (16, 16), (8, 8)]
    lat_np = I.bc1_pyramid(rng, sizes)
    uv_all = I.pixel_uv(96, 96, "tiled", jitter_rng=rng)
    for dims in ((14, 32, 32, 8), (14, 64, 64, 8), (14, 64, 64, 64, 8)):
        Ws, bs = I.xavier_mlp(rng, dims, bias="normal")
        lat, mlp = _gpu_case(lat_np, Ws, bs, I.PAPER_SHIFT)
        olat, omlp = _oracle_case(lat_np, Ws, bs, I.PAPER_SHIFT)
        packed = None
        if compute == "fp8":
            packed = ntc.pack(mlp, "fp8", act_amax=ntc.calibrate_fp8(lat, mlp, torch.from_numpy(uv_all).cuda()))
        for n in (1, 63, 65, 255, 257, 511, 513, 1025, 4099):
            uv = np.ascontiguousarray(uv_all[:n])
            out = torch.full((n + 5, dims[-1]), -3.0, device="cuda")
            ntc.decode(lat, mlp, torch.from_numpy(uv).cuda(), compute=compute, packed=packed, out=out[:n])
            got = out.cpu().numpy()
            assert np.all(got[n:] == -3.0), (dims, n)
            err = np.abs(got[:n].astype(np.float64) - O.decode(olat, omlp, uv))
            assert np.all(err <= tol), (dims, n, float(err.max()))


@pytest.mark.parametrize("dims,sizes,address,n", [
    ((14, 64, 64, 64, 8), [(64, 64), (32, 32), (16, 16), (8, 8)], "clamp", 1),
    ((14, 64, 64, 64, 64, 9), [(64, 64), (32, 32), (16, 16), (8, 8)], "clamp", 65),
    ((14, 32, 32, 8), [(64, 64), (32, 32), (16, 16), (8, 8)], "wrap", 127),
    ((11, 16, 3), [(64, 32), (32, 16), (16, 8)], "clamp", 129),
    ((5, 64, 16), [(32, 32)], "wrap", 4099),
    ((8, 32, 32, 32, 12), [(1024, 1024), (512, 512)], "clamp", 256 * 12 * 128 - 1),  # 64-pixel spans, then 128
    ((8, 32, 32, 32, 12), [(1024, 1024), (512, 512)], "clamp", 256 * 12 * 128 + 65),
])
@pytest.mark.parametrize("order", ["rows", "random"])
def test_f32_split_shapes(dims, sizes, address, n, order):
    """FP32 decode over the tails of 32-pixel tiles and 64- and 128-pixel
    spans, staged and direct texels, every network width and depth class:
    FP32 out within 1e-5 relative of the oracle, nothing written past the end,
    FP16 out within FP16 rounding."""
    ntc = _ntc()
    rng = np.random.default_rng(n + len(dims))
    lat_np = I.bc1_pyramid(rng, sizes)
    Ws, bs = I.xavier_mlp(rng, dims, bias="normal")
    shift = I.PAPER_SHIFT[:len(sizes)]
    if order == "rows":
        k = np.arange(n)
        uv = np.stack([(k % 700 + 0.5) / 700, (k // 700 + 0.5) / 600], 1).astype(np.float32)
    else:
        uv = (rng.random((n, 2)) * 1.4 - 0.2).astype(np.float32)
    lat = ntc.Latents(lat_np, shift=shift, address=address)
    mlp = ntc.Mlp(Ws, bs)
    ref = O.decode(O.Latents(lat_np, shift=shift, address=O.WRAP if address == "wrap" else O.CLAMP), O.Mlp(Ws, bs), uv)
    buf = torch.full((n + 4, dims[-1]), 7.0, device="cuda")
    ntc.decode(lat, mlp, torch.from_numpy(uv).cuda(), compute="f32", out=buf[:n])
    out = buf.cpu().numpy()
    assert np.all(out[n:] == 7.0)
    assert np.all(np.abs(out[:n] - ref) <= TOL_F32_REL * np.abs(ref))
    o16 = ntc.decode(lat, mlp, torch.from_numpy(uv).cuda(), compute="f32", out_dtype=torch.float16).cpu().numpy()
    assert np.all(np.abs(o16.astype(np.float64) - ref) <= 2.0 ** -11 * np.abs(ref) + 1e-7)


@pytest.mark.parametrize("fmt", ["bc1", "f32"])
@pytest.mark.parametrize("scale", [1.0, 2.0 ** 60, 2.0 ** 100, 2.0 ** 122, 2.0 ** -60, 2.0 ** -115])
def test_f32_split_range(scale, fmt):
    """FP32 decode of networks whose hidden activations are scaled by `scale`
    (undone by the next layer: the function stays the same): the largest
    leave the range in which numbers are split and take the FP32 matrix
    products, the smallest have parts below the normal range. Tolerance as
    for any FP32 decode."""
    ntc = _ntc()
    rng = np.random.default_rng(61)
    sizes = [(64, 64), (32, 32), (16, 16), (8, 8)]
    lat_np = I.bc1_pyramid(rng, sizes) if fmt == "bc1" else I.f32_pyramid(rng, sizes)
    Ws, bs = I.xavier_mlp(rng, (14, 64, 64, 8), bias="normal")
    Ws[0], bs[0] = (Ws[0] * np.float32(scale)), (bs[0] * np.float32(scale))
    Ws[1] = Ws[1] / np.float32(scale)
    uv = rng.random((40000, 2)).astype(np.float32)
    lat, mlp = _gpu_case(lat_np, Ws, bs, I.PAPER_SHIFT)
    out = ntc.decode(lat, mlp, torch.from_numpy(uv).cuda(), compute="f32").cpu().numpy()
    olat, omlp = _oracle_case(lat_np, Ws, bs, I.PAPER_SHIFT)
    ref = O.decode(olat, omlp, uv)
    assert np.all(np.abs(out - ref) <= TOL_F32_REL * np.abs(ref))


def test_f32_split_pixels_do_not_depend_on_neighbours():
    """Pixels with coordinates beyond the split range (and infinite or NaN
    latents) among others: the others equal a launch without them bit for bit,
    and the finite ones match the oracle."""
    ntc = _ntc()
    rng = np.random.default_rng(62)
    lat_np = I.f32_pyramid(rng, [(64, 64), (32, 32)])
    lat_np[0][5, 7] = np.inf
    lat_np[1][20, 3] = np.nan
    Ws, bs = I.xavier_mlp(rng, (8, 64, 64, 8), bias="normal")
    Ws[0][:, 6:] *= np.float32(1e-6)
    uv = rng.random((70000, 2)).astype(np.float32)
    far = uv.copy()
    at = rng.choice(uv.shape[0], 500, replace=False)
    far[at] *= np.float32(2.0e6)
    keep = np.ones(uv.shape[0], bool)
    keep[at] = False
    lat, mlp = _gpu_case(lat_np, Ws, bs, I.PAPER_SHIFT[:2])
    a = ntc.decode(lat, mlp, torch.from_numpy(uv).cuda(), compute="f32").cpu().numpy()
    b = ntc.decode(lat, mlp, torch.from_numpy(far).cuda(), compute="f32").cpu().numpy()
    assert np.array_equal(a[keep], b[keep], equal_nan=True)
    ref = O.decode(O.Latents(lat_np, shift=I.PAPER_SHIFT[:2]), O.Mlp(Ws, bs), far)
    fin = at[np.isfinite(O.features(O.Latents(lat_np, shift=I.PAPER_SHIFT[:2]), far[at])).all(1)]
    assert fin.size > 400
    assert np.all(np.abs(b[fin] - ref[fin]) <= TOL_F32_REL * np.abs(ref[fin]) + 1e-6)


@pytest.mark.parametrize("compute", ["f16", "bf16", "fp8", "f32"])
@pytest.mark.parametrize("sizes,scale,offset", [
    ([(64, 64), (32, 32), (16, 16), (8, 8)], 3.0, -1.0),       # spans across the edges, several periods
    ([(64, 32), (32, 16), (16, 8), (4, 4)], 0.3, 0.85),        # footprints over one edge
    ([(128, 128), (64, 64), (8, 8), (4, 4)], 40.0, -20.0),     # footprints wider than the small levels, or not staged
    ([(64, 64), (32, 32), (16, 16), (8, 8)], 1.0, 30000.0),    # far from the origin
    ([(64, 64), (32, 32), (16, 16), (8, 8)], 1.0e5, -4.0e4),   # positions past the staged range
])
def test_wrap_staged_equals_direct(compute, sizes, scale, offset):
    """Wrap addressing: coherent pixels (footprints staged before wrapping)
    give bit for bit what the same pixels give with the smallest staging
    capacity and in shuffled order (direct fetches), over edges, several
    periods, levels smaller than a footprint, coordinates far out and NaN."""
    ntc = _ntc()
    rng = np.random.default_rng(71)
    lat_np = I.bc1_pyramid(rng, sizes)
    Ws, bs = I.xavier_mlp(rng, (14, 32, 32, 9), bias="normal")
    Ws[0][:, 12:] *= np.float32(1.0 / max(1.0, abs(offset) + scale))
    lat = ntc.Latents(lat_np, shift=I.PAPER_SHIFT, address="wrap")
    mlp = ntc.Mlp(Ws, bs)
    w, h = 333, 61
    k = np.arange(w * h)
    uv = (np.stack([(k % w + 0.5) / w, (k // w + 0.5) / w], 1) * scale + offset).astype(np.float32)
    uv[5000] = np.nan
    uv[9000, 1] = np.inf
    amax = ntc.calibrate_fp8(lat, mlp, torch.rand((4096, 2), device="cuda")) if compute == "fp8" else None
    packed = ntc.pack(mlp, compute, act_amax=amax)
    t = torch.from_numpy(uv).cuda()
    a = ntc.decode(lat, mlp, t, compute=compute, packed=packed).cpu().numpy()
    fin = np.isfinite(uv).all(1)
    perm = rng.permutation(w * h)
    b = ntc.decode(lat, mlp, t[torch.from_numpy(perm).cuda()].contiguous(), compute=compute, packed=packed).cpu().numpy()
    assert np.array_equal(a[perm][fin[perm]], b[fin[perm]])
    if compute != "f32":
        c = ntc.decode(lat, mlp, t, compute=compute, packed=packed, cfg=ntc.tile_cfg(stage_capacity=64)).cpu().numpy()
        assert np.array_equal(a[fin], c[fin])
    # FP32 coordinates of this size carry the position to a fraction of a texel only as far as scale and offset allow
    if abs(offset) + scale <= 64.0 and compute in ("f32", "f16"):
        ref = O.decode(O.Latents(lat_np, shift=I.PAPER_SHIFT, address=O.WRAP), O.Mlp(Ws, bs), uv[fin])
        assert np.max(np.abs(a[fin] - ref)) <= (TOL_F16_ABS if compute == "f16" else 1e-5)


# Batches with spans of one tile (less than half of a first or second pass of
# the waves with long ones) and with long spans: a pixel does not depend on
# its span, so pieces equal the whole.
@pytest.mark.parametrize("compute", ["f16", "bf16", "fp8"])
@pytest.mark.parametrize("dims", [(14, 64, 64, 64, 8), (14, 32, 32, 5), (14, 16, 9)])
def test_short_batches_equal_long(compute, dims):
    ntc = _ntc()
    rng = np.random.default_rng(len(dims) + dims[-1])
    lat = ntc.Latents(I.bc1_pyramid(rng, [(64, 64), (32, 32), (16, 16), (8, 8)]), shift=I.PAPER_SHIFT)
    mlp = ntc.Mlp(*I.xavier_mlp(rng, dims, bias="normal"))
    n = 64 * 8 * torch.cuda.get_device_properties(0).multi_processor_count * 16 + 17  # long spans
    i = torch.arange(n, device="cuda")
    uv = torch.stack([(i % 1013) / 1013.0, (i // 1013) / 1100.0], 1).float()
    uv[-3000:] = torch.rand((3000, 2), generator=torch.Generator().manual_seed(1)).cuda() * 1.2 - 0.1
    uv = uv.contiguous()
    amax = ntc.calibrate_fp8(lat, mlp, uv[:65536].contiguous()) if compute == "fp8" else None
    packed = ntc.pack(mlp, compute, act_amax=amax)

    def run(a, b, dt=torch.float32):
        return ntc.decode(lat, mlp, uv[a:b].contiguous(), compute=compute, packed=packed, out_dtype=dt)

    whole, half = run(0, n), run(0, n, torch.float16)
    w = n // 16  # a tile a wave
    for a, b in ((0, 1), (5, 68), (64, 128), (1000, 1065), (0, w), (3 * w, 8 * w - 40), (w, 6 * w + 9), (0, 9 * w),
                 (n - 4000, n)):
        print(f"[short] {compute} {dims} {a}:{b}", flush=True)
        assert torch.equal(whole[a:b], run(a, b)), (a, b)
        assert torch.equal(half[a:b], run(a, b, torch.float16)), (a, b)


@pytest.mark.parametrize("dims,n", [((11, 32, 32, 32, 32, 4), 300), ((8, 64, 64, 64, 64, 8), 5000),
                                    ((8, 64, 64, 8), 70000)])
def test_f32_unused_levels_add_nothing(dims, n):
    """FP32 decode of fewer than four float levels whose first texels are not
    finite: pixels that do not sample them match the oracle."""
    ntc = _ntc()
    rng = np.random.default_rng(n)
    levels = (dims[0] - 2) // 3
    lat_np = I.f32_pyramid(rng, [(64, 64), (32, 32), (16, 16)][:levels])
    lat_np[0][0, 0], lat_np[0][1, 1] = np.inf, np.nan
    Ws, bs = I.xavier_mlp(rng, dims, bias="normal")
    shift = I.PAPER_SHIFT[:levels]
    uv = (0.1 + 0.9 * rng.random((n, 2))).astype(np.float32)
    lat, mlp = _gpu_case(lat_np, Ws, bs, shift)
    out = ntc.decode(lat, mlp, torch.from_numpy(uv).cuda(), compute="f32").cpu().numpy()
    ref = O.decode(O.Latents(lat_np, shift=shift), O.Mlp(Ws, bs), uv)
    assert np.all(np.abs(out - ref) <= TOL_F32_REL * np.abs(ref))


@pytest.mark.parametrize("fmt", ["bc1", "f32"])
@pytest.mark.parametrize("layer", [0, 1])
@pytest.mark.parametrize("exponent", [-40, -80, -100, -110, -113, -118, -122, 110])
def test_f32_small_numbers(exponent, layer, fmt):
    """FP32 decode of networks with one hidden layer scaled by a power of two
    and the next by its reciprocal (exactly): the result is that of the plain
    network to FP32 accuracy, also where parts of the split numbers fall
    below the normal range. FP32 chains of 64 terms stay well below 2e-6."""
    ntc = _ntc()
    rng = np.random.default_rng(63)
    sizes = [(64, 64), (32, 32), (16, 16), (8, 8)]
    lat_np = I.bc1_pyramid(rng, sizes) if fmt == "bc1" else I.f32_pyramid(rng, sizes)
    Ws, bs = I.xavier_mlp(rng, (14, 64, 64, 64, 8), bias="normal")
    # weights of 12 significant bits, so that scaling into the subnormal range is exact
    Ws = [np.ldexp(np.rint(np.ldexp(w, 12)), -12).astype(np.float32) for w in Ws]
    bs = [np.ldexp(np.rint(np.ldexp(b, 12)), -12).astype(np.float32) for b in bs]
    uv = rng.random((40000, 2)).astype(np.float32)
    olat, omlp = _oracle_case(lat_np, Ws, bs, I.PAPER_SHIFT)
    ref = O.decode(olat, omlp, uv)
    Ws[layer], bs[layer] = np.ldexp(Ws[layer], exponent), np.ldexp(bs[layer], exponent)
    Ws[layer + 1] = np.ldexp(Ws[layer + 1], -exponent)
    lat, mlp = _gpu_case(lat_np, Ws, bs, I.PAPER_SHIFT)
    out = ntc.decode(lat, mlp, torch.from_numpy(uv).cuda(), compute="f32").cpu().numpy()
    err = np.max(np.abs(out - ref) / ref)
    print(f"[small numbers] {fmt} layer {layer} 2^{exponent}: {err:.1e}", flush=True)
    assert err <= 2e-6


@pytest.mark.parametrize("dims,address", [((14, 16, 9), "clamp"), ((11, 32, 32, 3), "wrap"), ((14, 64, 16), "clamp"),
                                          ((8, 32, 32, 32, 32, 5), "wrap"), ((5, 16, 16, 16, 4), "clamp"),
                                          ((14, 64, 64, 64, 64, 8), "clamp")])
@pytest.mark.parametrize("fmt", ["bc1", "f32"])
@pytest.mark.parametrize("whole", [True, False])
def test_f32_second_walk_shapes(dims, address, fmt, whole):
    """The walk over pixels that may not be split, over every width and depth
    class and the tails of its tiles: all pixels (a hidden layer scaled by
    2^122, the next by its reciprocal) and single pixels with far
    coordinates; nothing is written past the end."""
    ntc = _ntc()
    rng = np.random.default_rng(len(dims) * 100 + dims[1])
    levels = (dims[0] - 2) // 3
    sizes = [(64, 32), (32, 32), (16, 8), (8, 8)][:levels]
    lat_np = I.bc1_pyramid(rng, sizes) if fmt == "bc1" else I.f32_pyramid(rng, sizes)
    Ws, bs = I.xavier_mlp(rng, dims, bias="normal")
    if whole:
        Ws[0], bs[0], Ws[1] = np.ldexp(Ws[0], 122), np.ldexp(bs[0], 122), np.ldexp(Ws[1], -122)
    else:
        Ws[0][:, -2:] *= np.float32(1e-7)
    shift = I.PAPER_SHIFT[:levels]
    lat, mlp = _gpu_case(lat_np, Ws, bs, shift, address)
    # short batches of float latents with up to four layers take another kernel
    ns = (1, 65, 4099) if fmt == "bc1" or len(dims) > 5 else (2 ** 21 // dims[1] + 65,)
    for n in ns:
        uv = (rng.random((n, 2)) * 1.4 - 0.2).astype(np.float32)
        if not whole:
            uv[rng.choice(n, max(1, n // 50), replace=False)] += np.float32(2.0 ** 21)
        # sampling positions are limited to 2^24 texels: under wrap addressing such a pixel's texels are not the oracle's
        near = np.abs(uv).max(1) < 2.0 ** 20 if address == "wrap" else np.ones(n, bool)
        buf = torch.full((n + 4, dims[-1]), 7.0, device="cuda")
        ntc.decode(lat, mlp, torch.from_numpy(uv).cuda(), compute="f32", out=buf[:n])
        out = buf.cpu().numpy()
        assert np.all(out[n:] == 7.0)
        olat, omlp = _oracle_case(lat_np, Ws, bs, shift, address)
        ref = O.decode(olat, omlp, uv)
        assert np.isfinite(out).all()
        assert np.all((np.abs(out[:n] - ref) <= TOL_F32_REL * np.abs(ref))[near]), n


@pytest.mark.parametrize("compute,dims", [("f16", (14, 64, 64, 64, 8)), ("f16", (14, 32, 32, 5)), ("bf16", (14, 16, 9))])
def test_launched_waves_do_not_change_results(compute, dims):
    """waves_per_cu decides the launch and the span length, not the result."""
    ntc = _ntc()
    rng = np.random.default_rng(dims[-1])
    lat = ntc.Latents(I.bc1_pyramid(rng, [(64, 64), (32, 32), (16, 16), (8, 8)]), shift=I.PAPER_SHIFT)
    mlp = ntc.Mlp(*I.xavier_mlp(rng, dims, bias="normal"))
    packed = ntc.pack(mlp, compute)
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    for tiles in (8 * cus + 1, 8 * cus * 4, 8 * cus * 5 + 3, 8 * cus * 9 + 1):
        i = torch.arange(64 * tiles - 7, device="cuda")
        uv = torch.stack([(i % 1013) / 1013.0, (i // 1013) / 1200.0], 1).float().contiguous()
        ref = ntc.decode(lat, mlp, uv, compute=compute, packed=packed)
        for w in (1, 3, 16, 64, 1024):
            got = ntc.decode(lat, mlp, uv, compute=compute, packed=packed, cfg=ntc.tile_cfg(waves_per_cu=w))
            assert torch.equal(ref, got), (tiles, w)


# One long span per wave, then single tiles: first tile after the spans, last
# waves without one, two per wave, a last tile that is not full, and the batch
# sizes next to where that begins and ends.
@pytest.mark.parametrize("compute,dims", [("f16", (14, 16, 8)), ("f16", (14, 64, 64, 5)), ("bf16", (14, 32, 32, 9)),
                                          ("fp8", (14, 32, 32, 32, 32, 8))])
def test_long_span_then_tiles_equals_long(compute, dims):
    ntc = _ntc()
    rng = np.random.default_rng(dims[-1])
    lat = ntc.Latents(I.bc1_pyramid(rng, [(64, 64), (32, 32), (16, 16), (8, 8)]), shift=I.PAPER_SHIFT)
    mlp = ntc.Mlp(*I.xavier_mlp(rng, dims, bias="normal"))
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    amax = ntc.calibrate_fp8(lat, mlp, torch.rand((65536, 2), device="cuda")) if compute == "fp8" else None
    packed = ntc.pack(mlp, compute, act_amax=amax)
    for wpc in (1, 8):
        waves = cus * wpc
        n = 64 * 8 * waves * 16 + 5  # long spans alone
        i = torch.arange(n, device="cuda")
        uv = torch.stack([(i % 1013) / 1013.0, (i // 1013) / (n / 1013.0)], 1).float().contiguous()
        cfg = ntc.tile_cfg(waves_per_cu=wpc)
        whole = ntc.decode(lat, mlp, uv, compute=compute, packed=packed, cfg=cfg)
        for px in (64 * 8 * waves, 64 * 8 * waves + 1, 64 * (9 * waves - 1) + 63, 64 * 9 * waves, 64 * 9 * waves + 64,
                   64 * 12 * waves, 64 * 12 * waves + 1):
            buf = torch.full((px + 4, dims[-1]), 7.0, device="cuda")
            ntc.decode(lat, mlp, uv[:px], compute=compute, packed=packed, cfg=cfg, out=buf[:px])
            assert torch.equal(whole[:px], buf[:px]), (wpc, px)
            assert bool((buf[px:] == 7.0).all())
