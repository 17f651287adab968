"""Frame classification (ntc_classify; Sec. 4, Algorithm 1) and the frame
decode it feeds, against the oracle (oracle/classify.py, FP64 decode).
Lists, offsets and tile classes are integer results in a fixed order:
bit-exact."""
import numpy as np
import pytest
import torch

import ntc_inputs as I
import oracle as O
from oracle import classify as C

pytestmark = pytest.mark.gpu


def _ntc():
    import paper_2506_06040_amd as ntc
    return ntc


FRAMES = [
    dict(w=64, h=32, n=3, noise=0.0, seed=1),
    dict(w=37, h=22, n=5, noise=0.05, seed=2),
    dict(w=256, h=128, n=40, noise=0.02, seed=3),
    dict(w=200, h=120, n=1, noise=0.0, seed=4),
    dict(w=1024, h=512, n=64, noise=0.01, seed=5),
    dict(w=9, h=5, n=2, noise=0.0, seed=6, background=1.0),
    dict(w=130, h=66, n=300, noise=0.3, seed=7),
]


@pytest.mark.parametrize("f", FRAMES, ids=lambda f: f"{f['w']}x{f['h']}_m{f['n']}")
def test_classify_bitexact(f):
    ntc = _ntc()
    rng = np.random.default_rng(f["seed"])
    mat = I.material_frame(rng, f["w"], f["h"], f["n"], noise=f["noise"], background=f.get("background", 0.15))
    print(f"[classify] {f}", flush=True)
    lst, off, simple, tcls = ntc.classify(torch.from_numpy(mat).cuda(), f["n"])
    olst, ooff, osimple, otcls = C.classify(mat, f["n"])
    assert np.array_equal(off.cpu().numpy(), ooff)
    assert np.array_equal(simple.cpu().numpy(), osimple)
    assert np.array_equal(tcls.cpu().numpy(), otcls)
    assert np.array_equal(lst.cpu().numpy(), olst)
    # the same input gives the same lists
    lst2 = ntc.classify(torch.from_numpy(mat).cuda(), f["n"])[0]
    assert torch.equal(lst, lst2)


# Both widths of the walk (up to 1024 materials eight wavefronts share a chunk
# of 128 tiles), a last chunk of one tile, of one wavefront's and of all but
# one wavefront's tiles, frames of noise alone.
@pytest.mark.parametrize("w,h,n,noise", [(8, 4 * 129, 2, 0.5), (8, 4 * 144, 70, 1.0), (1024, 4 * 7 - 1, 1024, 0.1),
                                         (1024, 4 * 7 - 1, 1025, 0.1), (333, 77, 4096, 1.0)])
def test_classify_chunk_shares(w, h, n, noise):
    ntc = _ntc()
    mat = I.material_frame(np.random.default_rng(w + h + n), w, h, n, noise=noise)
    olst, ooff, osimple, otcls = C.classify(mat, n)
    for classes in (True, False):
        lst, off, simple, tcls = ntc.classify(torch.from_numpy(mat).cuda(), n, tile_class=classes)
        assert np.array_equal(off.cpu().numpy(), ooff)
        assert np.array_equal(simple.cpu().numpy(), osimple)
        assert np.array_equal(lst.cpu().numpy(), olst)
        assert tcls is None if not classes else np.array_equal(tcls.cpu().numpy(), otcls)


def test_gather_and_scatter():
    ntc = _ntc()
    rng = np.random.default_rng(8)
    h, w = 48, 80
    uv_img = rng.random((h, w, 2)).astype(np.float32)
    idx = rng.permutation(h * w)[:1000].astype(np.int32)
    uv = ntc.gather_uv(torch.from_numpy(uv_img).cuda(), torch.from_numpy(idx).cuda()).cpu().numpy()
    assert np.array_equal(uv, uv_img.reshape(-1, 2)[idx])
    for dt in (torch.float32, torch.float16):
        rows = torch.from_numpy(rng.random((1000, 9)).astype(np.float32)).to(dt).cuda()
        img = torch.zeros((h, w, 9), dtype=dt, device="cuda")
        ntc.scatter_rows(rows, torch.from_numpy(idx).cuda(), img)
        ref = np.zeros((h * w, 9), np.float32)
        ref[idx] = rows.float().cpu().numpy()
        assert np.array_equal(img.float().cpu().numpy().reshape(-1, 9), ref)


def test_frame_decode_equals_per_material_and_oracle():
    ntc = _ntc()
    rng = np.random.default_rng(9)
    h, w, n_mats = 192, 256, 6
    mat = I.material_frame(rng, w, h, n_mats, noise=0.02)
    uv_img = I.pixel_uv(w, h).reshape(h, w, 2)
    dims = [(14, 64, 64, 64, 8), (14, 32, 32, 8), (14, 64, 8), (14, 16, 16, 16, 8), (14, 64, 64, 8), (14, 32, 8)]
    mats, omats = [], []
    for m in range(n_mats):
        lat_np = I.bc1_pyramid(rng, [(128, 128), (64, 64), (32, 32), (16, 16)])
        Ws, bs = I.xavier_mlp(rng, dims[m], bias="normal")
        mats.append((ntc.Latents(lat_np, shift=I.PAPER_SHIFT), ntc.Mlp(Ws, bs)))
        omats.append((O.Latents(lat_np, shift=I.PAPER_SHIFT), O.Mlp(Ws, bs)))
    fd = ntc.FrameDecoder(mats)
    mat_t = torch.from_numpy(mat).cuda()
    uv_t = torch.from_numpy(np.ascontiguousarray(uv_img)).cuda()
    out_t = fd.decode(mat_t, uv_t)
    # the decode through the pixel lists equals gather + decode + scatter
    assert torch.equal(out_t, fd.decode(mat_t, uv_t, indexed=False))
    out = out_t.cpu().numpy().reshape(-1, 8)
    lst, off, _, _ = ntc.classify(mat_t, n_mats)
    lst, off = lst.cpu().numpy(), off.cpu().numpy()
    flat_uv = uv_img.reshape(-1, 2)
    invalid = np.nonzero(mat.reshape(-1) >= n_mats)[0]
    assert np.all(out[invalid] == 0.0)
    for m, ((lat, mlp), (olat, omlp)) in enumerate(zip(mats, omats)):
        pix = lst[off[m]:off[m + 1]]
        if pix.size == 0:
            continue
        single = ntc.decode(lat, mlp, torch.from_numpy(flat_uv[pix]).cuda(), compute="f16").cpu().numpy()
        assert np.array_equal(out[pix], single), m
        ref = O.decode(olat, omlp, flat_uv[pix])
        err = np.abs(out[pix] - ref).max()
        print(f"[frame decode] material {m}: {pix.size} px, max err {err:.2e}", flush=True)
        assert err <= 2e-3, m


def test_batched_indexed_ignores_invalid_indices():
    """Indices outside the image read uv (0, 0) and write nothing; valid ones
    equal the plain decode of the same uv."""
    ntc = _ntc()
    rng = np.random.default_rng(10)
    h, w = 64, 96
    lat_np = I.bc1_pyramid(rng, [(64, 64), (32, 32), (16, 16), (8, 8)])
    Ws, bs = I.xavier_mlp(rng, (14, 32, 32, 8), bias="normal")
    lat, mlp = ntc.Latents(lat_np, shift=I.PAPER_SHIFT), ntc.Mlp(Ws, bs)
    uv_img = torch.from_numpy(rng.random((h * w, 2)).astype(np.float32)).cuda()
    idx = rng.permutation(h * w)[:2000].astype(np.int32)
    idx[::97] = -1
    idx[5::97] = h * w + 3
    out = torch.full((h * w, 8), 7.0, device="cuda")
    m = ntc.Material(lat, mlp, uv_img, out=out, pixel_index=torch.from_numpy(idx).cuda())
    ntc.BatchPlan([m]).launch()
    torch.cuda.synchronize()
    good = idx[(idx >= 0) & (idx < h * w)]
    ref = ntc.decode(lat, mlp, uv_img[torch.from_numpy(good).long().cuda()].contiguous(), compute="f16")
    got = out.cpu().numpy()
    assert np.array_equal(got[good], ref.cpu().numpy())
    untouched = np.setdiff1d(np.arange(h * w), good)
    assert np.all(got[untouched] == 7.0)


# The plan built on the device against the one built on the host (a cfg of
# one's own) and against gather, decode and scatter: every MLP shape, frames
# with fewer tiles than waves, of one pixel, without neural pixels, with more
# materials than pixels, FP16 outputs and pixels that keep their value.
@pytest.mark.parametrize("w,h,n,noise,bg,dt", [
    (256, 192, 9, 0.02, 0.15, torch.float32), (1024, 512, 40, 0.01, 0.1, torch.float16),
    (1, 1, 1, 0.0, 0.0, torch.float32), (9, 5, 3, 1.0, 1.0, torch.float32), (37, 22, 300, 1.0, 0.2, torch.float32),
    (640, 360, 2, 0.0, 0.0, torch.float32)])
def test_frame_plan_on_device_equals_host_plan(w, h, n, noise, bg, dt):
    ntc = _ntc()
    rng = np.random.default_rng(w + n)
    mat = I.material_frame(rng, w, h, n, noise=noise, background=bg)
    mats = []
    for m in range(n):
        lat_np = I.bc1_pyramid(rng, [(32, 32), (16, 16), (8, 8), (4, 4)])
        dims = (14,) + ((16, 32, 64)[m % 3],) * (1 + m // 3 % 3) + (8,)
        mats.append((ntc.Latents(lat_np, shift=I.PAPER_SHIFT), ntc.Mlp(*I.xavier_mlp(rng, dims, bias="normal"))))
    mat_t = torch.from_numpy(mat).cuda()
    uv = torch.from_numpy(rng.random((h, w, 2)).astype(np.float32)).cuda()
    dev = ntc.FrameDecoder(mats, out_dtype=dt)
    host = ntc.FrameDecoder(mats, cfg=ntc.batch_cfg(item_pixels=128, n_cus=8), out_dtype=dt)

    def image(fd, **kw):
        return fd.decode(mat_t, uv, out=torch.full((h, w, 8), 7.0, dtype=dt, device="cuda"), **kw)

    ref = image(host)
    assert torch.equal(ref, image(dev, indexed=False))
    assert torch.equal(ref, image(dev))
    assert torch.equal(ref, image(dev))  # the table of the first frame
    assert bool((ref.cpu().numpy()[mat >= n] == 7.0).all())
    # other weights in the decoder's list of images
    dev.packed[0] = ntc.pack(ntc.Mlp(*I.xavier_mlp(rng, [int(d) for d in mats[0][1].dims], bias="normal")), "f16")
    host.packed[0] = dev.packed[0]
    assert torch.equal(image(host), image(dev))
    # other materials, on another stream
    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(s):
        dev.materials.reverse(), dev.packed.reverse(), host.materials.reverse(), host.packed.reverse()
        assert torch.equal(image(host), image(dev))
    torch.cuda.current_stream().wait_stream(s)


def test_frame_decode_rejects_as_before():
    ntc = _ntc()
    rng = np.random.default_rng(3)
    lat = ntc.Latents(I.bc1_pyramid(rng, [(16, 16), (8, 8)]), shift=I.PAPER_SHIFT[:2])
    deep = ntc.Mlp(*I.xavier_mlp(rng, (8, 16, 16, 16, 16, 4), bias="normal"))
    fd = ntc.FrameDecoder([(lat, deep)])  # five layers: not in a batch
    uv = torch.zeros((8, 8, 2), device="cuda")
    with pytest.raises(ntc.NtcError):
        fd.decode(torch.zeros((8, 8), dtype=torch.int16, device="cuda"), uv)
    assert not fd.decode(torch.full((8, 8), 5, dtype=torch.int16, device="cuda"), uv).any()
    fd = ntc.FrameDecoder([(lat, ntc.Mlp(*I.xavier_mlp(rng, (8, 16, 4), bias="normal")))])
    with pytest.raises(ValueError):
        fd.decode(torch.zeros((8, 8), dtype=torch.int32, device="cuda"), uv)
    with pytest.raises(ValueError):
        fd.decode(torch.zeros((8, 8), dtype=torch.int16, device="cuda"), uv.cpu())
    with pytest.raises(ntc.NtcError):  # misaligned uv
        fd.decode(torch.zeros((8, 8), dtype=torch.int16, device="cuda"),
                  torch.zeros(129, device="cuda")[1:].reshape(8, 8, 2))


@pytest.mark.parametrize("view", ["columns", "expanded"])
def test_frame_decode_rejects_strided_uv(view):
    """Coordinates that are not adjacent pairs: ValueError where there is
    something to decode, nothing to do (and no error) where there is not."""
    ntc = _ntc()
    rng = np.random.default_rng(4)
    lat = ntc.Latents(I.bc1_pyramid(rng, [(16, 16), (8, 8)]), shift=I.PAPER_SHIFT[:2])
    fd = ntc.FrameDecoder([(lat, ntc.Mlp(*I.xavier_mlp(rng, (8, 16, 4), bias="normal")))])
    uv = torch.rand((8, 8, 4), device="cuda")[..., :2] if view == "columns" else torch.rand((1, 1, 2), device="cuda").expand(8, 8, 2)
    assert not uv.reshape(-1, 2).is_contiguous()
    with pytest.raises(ValueError):
        fd.decode(torch.zeros((8, 8), dtype=torch.int16, device="cuda"), uv)
    assert not fd.decode(torch.full((8, 8), 5, dtype=torch.int16, device="cuda"), uv).any()
    # a transposed image is copied into pairs
    t = torch.rand((8, 8, 2), device="cuda").transpose(0, 1)
    ids = torch.zeros((8, 8), dtype=torch.int16, device="cuda")
    assert torch.equal(fd.decode(ids, t), fd.decode(ids, t.contiguous()))


def test_frame_without_neural_pixels_keeps_any_output_type():
    ntc = _ntc()
    rng = np.random.default_rng(5)
    lat = ntc.Latents(I.bc1_pyramid(rng, [(16, 16), (8, 8)]), shift=I.PAPER_SHIFT[:2])
    fd = ntc.FrameDecoder([(lat, ntc.Mlp(*I.xavier_mlp(rng, (8, 16, 4), bias="normal")))], out_dtype=torch.bfloat16)
    uv = torch.rand((8, 8, 2), device="cuda")
    assert not fd.decode(torch.full((8, 8), 5, dtype=torch.int16, device="cuda"), uv).any()
    with pytest.raises(KeyError):
        fd.decode(torch.zeros((8, 8), dtype=torch.int16, device="cuda"), uv)


def test_frame_decode_captured():
    """A captured frame decode follows its inputs and keeps its materials when
    the decoder has gone on to others, over several replays with eager work
    between them."""
    ntc = _ntc()
    rng = np.random.default_rng(6)
    h, w = 72, 104

    def materials(n):
        return [(ntc.Latents(I.bc1_pyramid(rng, [(32, 32), (16, 16)]), shift=I.PAPER_SHIFT[:2]),
                 ntc.Mlp(*I.xavier_mlp(rng, (8, (16, 32, 64)[m % 3], 4), bias="normal"))) for m in range(n)]

    first, second = materials(5), materials(5)
    fd, ref = ntc.FrameDecoder(first), ntc.FrameDecoder(first)
    packed = list(fd.packed)
    frames = [(torch.from_numpy(I.material_frame(rng, w, h, 5, noise=0.02)).cuda(),
               torch.from_numpy(rng.random((h, w, 2)).astype(np.float32)).cuda()) for _ in range(3)]
    ids, uv = frames[0][0].clone(), frames[0][1].clone()
    out = torch.zeros((h, w, 4), device="cuda")
    fd.decode(ids, uv, out=out)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        fd.decode(ids, uv, out=out)
    table = fd._table[2]
    fd.materials, fd.packed = second, [ntc.pack(m, "f16") for _, m in second]
    fd.decode(*frames[0])
    assert fd._table[2] is not table and fd._captured == [table]
    for i in range(6):
        ids.copy_(frames[i % 3][0]), uv.copy_(frames[i % 3][1])
        out.zero_()
        torch.full((1 << 20,), 255, dtype=torch.uint8, device="cuda")
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, ref.decode(*frames[i % 3])), i
    del packed
