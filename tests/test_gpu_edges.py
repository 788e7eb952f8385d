"""Sizes at the edges of the kernels' tiles, groups and dispatch rules, against the oracle."""
import numpy as np
import pytest

import oracle
from paper_2509_09679_amd import synth

pytestmark = pytest.mark.gpu
gu = pytest.importorskip("gpu_util")


@pytest.mark.parametrize("n,heads", [(2, 3), (64, 5), (128, 3), (256, 3), (512, 1), (8192, 2), (16384, 1)])
def test_plan_tables_at_the_group_sizes(n, heads):
    # plan_table_kernel: one group of all layers up to n = 128, low and high groups of unequal and equal size above;
    # the float32 path uses the forward and the transposed tables, the backward pass the sums' scales as well
    rows = 5
    x, th, dy = synth.small_case(n, rows, "f32", heads=heads, seed=300 + n, with_dy=True, outliers=0)
    x64, dy64 = synth.to_f64(x, "f32"), synth.to_f64(dy, "f32")
    gu.check_rotated(gu.run_transform(x, th, n, heads, "f32"), oracle.forward(x64, th, n, heads), "f32", f"fwd n={n}")
    gu.check_rotated(gu.run_transform(x, th, n, heads, "f32", inverse=True), oracle.inverse(x64, th, n, heads), "f32", f"inv n={n}")
    rdx, rdth, ab = oracle.backward(x64, dy64, th, n, heads)
    dx, dth = gu.run_bwd(x, dy, th, n, heads, "f32")
    gu.check_rotated(dx, rdx, "f32", f"dx n={n}")
    # with a handful of rows an angle's own products may nearly cancel: the bound is floored at the layer's median (the
    # seeded sweep states why)
    floor = np.median(ab, axis=2, keepdims=True)
    gu.check_dtheta(dth, rdth, np.maximum(ab, floor), what=f"dtheta n={n}")


@pytest.mark.parametrize("n,heads,rows,dtype", [(4096, 1, 1, "f16"), (4096, 2, 3, "f32"), (8192, 1, 1, "bf16"), (8192, 1, 2, "f32"),
                                                (8192, 2, 5, "f16"), (256, 16, 2, "f16"), (1024, 4, 3, "f32"), (2048, 1, 2, "bf16")])
@pytest.mark.parametrize("bits,group,sd", [(4, 128, "f16"), (2, 64, "f32"), (4, 256, "f16")])
def test_few_rows_through_every_transform_kernel(n, heads, rows, dtype, bits, group, sd):
    # the pipelines' fill and drain without a steady state in between, tables transposed through the row buffers that the
    # first rows then use, constants parked in LDS
    x, th, _ = synth.small_case(n, rows, dtype, heads=heads, seed=400 + n + rows)
    x64 = synth.to_f64(x, dtype)
    ref = oracle.forward(x64, th, n, heads)
    tag = f"n={n} H={heads} T={rows} {dtype}"
    gu.check_rotated(gu.run_transform(x, th, n, heads, dtype), ref, dtype, tag + " fwd")
    gu.check_rotated(gu.run_transform(x, th, n, heads, dtype, inverse=True), oracle.inverse(x64, th, n, heads), dtype, tag + " inv")
    codes, scales = gu.run_fwd_quant(x, th, n, heads, dtype, bits, group, sd)
    gu.check_fused_codes(codes, scales, ref, bits, group, sd, dtype, tag)
    c = oracle.unpack_codes(codes, bits)
    want = synth.cast_storage(oracle.dequantize(c, scales.astype(np.float32), group).astype(np.float64), dtype)
    u = np.uint16 if dtype != "f32" else np.uint32
    for want_y, want_hist in ((True, True), (True, False), (False, True)):
        yq, hist = gu.run_fwd_fakequant(x, th, n, heads, dtype, bits, group, sd, want_y=want_y, want_hist=want_hist)
        if want_y:
            np.testing.assert_array_equal(yq.view(u), want.view(u), err_msg=tag)
        if want_hist:
            np.testing.assert_array_equal(hist, oracle.bin_histogram(c, bits), err_msg=tag)


@pytest.mark.parametrize("n,heads,rows", [(64, 12, 5), (32, 3, 33), (128, 5, 7), (128, 33, 3), (8, 3, 200), (8, 257, 2), (16, 127, 3),
                                          (128, 9, 4), (128, 65, 1), (64, 1, 1), (8, 67, 40)])
@pytest.mark.parametrize("dtype", ["f16", "f32"])
def test_small_transforms_of_any_row_width(n, heads, rows, dtype):
    # small_tiling: idle lanes behind the last whole row of a workgroup, slices whose last one is short, one to four waves;
    # strided rows and every mode through the same tiling
    x, th, dy = synth.small_case(n, rows, dtype, heads=heads, seed=500 + n * heads + rows, with_dy=True, outliers=0)
    x64, dy64 = synth.to_f64(x, dtype), synth.to_f64(dy, dtype)
    ref = oracle.forward(x64, th, n, heads)
    tag = f"n={n} H={heads} T={rows} {dtype}"
    for pad in (0, 8):
        gu.check_rotated(gu.run_transform(x, th, n, heads, dtype, pad=pad), ref, dtype, tag + " fwd")
        gu.check_rotated(gu.run_transform(x, th, n, heads, dtype, inverse=True, pad=pad), oracle.inverse(x64, th, n, heads), dtype,
                         tag + " inv")
    for bits, group, sd in ((4, n, "f16"), (2, 8, "f32")):
        codes, scales = gu.run_fwd_quant(x, th, n, heads, dtype, bits, group, sd)
        gu.check_fused_codes(codes, scales, ref, bits, group, sd, dtype, tag)
        c = oracle.unpack_codes(codes, bits)
        want = synth.cast_storage(oracle.dequantize(c, scales.astype(np.float32), group).astype(np.float64), dtype)
        yq, hist = gu.run_fwd_fakequant(x, th, n, heads, dtype, bits, group, sd)
        u = np.uint16 if dtype != "f32" else np.uint32
        np.testing.assert_array_equal(yq.view(u), want.view(u), err_msg=tag)
        np.testing.assert_array_equal(hist, oracle.bin_histogram(c, bits), err_msg=tag)
    rdx, rdth, ab = oracle.backward(x64, dy64, th, n, heads)
    floor = np.median(ab, axis=2, keepdims=True)  # (few rows: as in the seeded sweep)
    for pad in (0, 8):
        dx, dth = gu.run_bwd(x, dy, th, n, heads, dtype, pad=pad)
        gu.check_rotated(dx, rdx, dtype, tag + " dx")
        gu.check_dtheta(dth, rdth, np.maximum(ab, floor), what=tag + " dtheta")


@pytest.mark.parametrize("n,heads,rows", [(4096, 1, 9), (8192, 1, 5), (1024, 2, 7), (2048, 1, 3), (128, 3, 33), (64, 12, 40), (8, 1, 600),
                                          (16384, 1, 2)])
@pytest.mark.parametrize("dtype", ["f16", "f32"])
def test_backward_of_flagged_plans_through_every_route(n, heads, rows, dtype):
    # angles of pi/2 in three layers drive the deferred scales out of range: the specialised kernels leave the batch to the
    # generic one and their second pass adds that kernel's partial sums (n < 4096: the fold kernel does)
    x, th, dy = synth.small_case(n, rows, dtype, heads=heads, seed=600 + n * heads, with_dy=True, outliers=0)
    th = th.copy()
    th[:, :3] = np.float32(np.pi / 2)
    x64, dy64 = synth.to_f64(x, dtype), synth.to_f64(dy, dtype)
    rdx, rdth, ab = oracle.backward(x64, dy64, th, n, heads)
    floor = np.median(ab, axis=2, keepdims=True)  # (few rows: as in the seeded sweep)
    dx, dth = gu.run_bwd(x, dy, th, n, heads, dtype)
    tag = f"n={n} H={heads} T={rows} {dtype}"
    gu.check_rotated(dx, rdx, dtype, tag + " dx")
    gu.check_dtheta(dth, rdth, np.maximum(ab, floor), what=tag + " dtheta")


@pytest.mark.parametrize("n,heads,rows", [(256, 1, 1), (256, 1, 17), (256, 1, 15 + 16 * 300), (256, 4, 5), (512, 1, 7), (512, 8, 3), (1024, 2, 3),
                                          (1024, 1, 1025), (2048, 1, 1), (2048, 1, 2563), (2048, 2, 3)])
@pytest.mark.parametrize("dtype", ["f16", "f32"])
def test_short_last_block_of_narrow_transforms(n, heads, rows, dtype):
    # a block of 4096 elements whose rows are not all there: their lanes read copies and store, count and pack nothing; every
    # mode, strided rows, in place, flagged plans, groups within a wave and across waves
    x, th, _ = synth.small_case(n, rows, dtype, heads=heads, seed=700 + n * heads + rows)
    x64 = synth.to_f64(x, dtype)
    flagged = th.copy()
    flagged[:, :3] = np.float32(np.pi / 2)
    for angles, tag in ((th, ""), (flagged, " flagged")):
        tag = f"n={n} H={heads} T={rows} {dtype}" + tag
        ref, back = oracle.forward(x64, angles, n, heads), oracle.inverse(x64, angles, n, heads)
        for pad, inplace in ((0, False), (8, False), (0, True)):
            gu.check_rotated(gu.run_transform(x, angles, n, heads, dtype, pad=pad, inplace=inplace), ref, dtype, tag + " fwd")
            gu.check_rotated(gu.run_transform(x, angles, n, heads, dtype, inverse=True, pad=pad, inplace=inplace), back, dtype, tag + " inv")
        for bits, group, sd in ((4, 128, "f16"), (2, n, "f32")):
            codes, scales = gu.run_fwd_quant(x, angles, n, heads, dtype, bits, group, sd)
            gu.check_fused_codes(codes, scales, ref, bits, group, sd, dtype, tag)
            c = oracle.unpack_codes(codes, bits)
            want = synth.cast_storage(oracle.dequantize(c, scales.astype(np.float32), group).astype(np.float64), dtype)
            u = np.uint16 if dtype != "f32" else np.uint32
            yq, hist = gu.run_fwd_fakequant(x, angles, n, heads, dtype, bits, group, sd)
            np.testing.assert_array_equal(yq.view(u), want.view(u), err_msg=tag)
            np.testing.assert_array_equal(hist, oracle.bin_histogram(c, bits), err_msg=tag)
            _, hist = gu.run_fwd_fakequant(x, angles, n, heads, dtype, bits, group, sd, want_y=False)
            np.testing.assert_array_equal(hist, oracle.bin_histogram(c, bits), err_msg=tag)


@pytest.mark.parametrize("n,heads,rows", [(8, 1, 300), (8, 3, 77), (16, 5, 40), (32, 3, 33), (64, 12, 700), (128, 1, 200), (128, 20, 60),
                                          (128, 32, 40), (8192, 1, 3), (8192, 2, 2)])
@pytest.mark.parametrize("dtype", ["f16", "bf16", "f32"])
def test_transforms_of_flagged_plans(n, heads, rows, dtype):
    # n = 8 .. 128: rotations held in registers, with idle lanes and several row groups per workgroup; n = 8192: the layers
    # through LDS, several pairs per thread at a time
    x, th, _ = synth.small_case(n, rows, dtype, heads=heads, seed=1000 + n * heads)
    th = th.copy()
    th[:, :3] = np.float32(np.pi / 2)
    x64 = synth.to_f64(x, dtype)
    tag = f"n={n} H={heads} T={rows} {dtype}"
    for pad in (0, 8):
        gu.check_rotated(gu.run_transform(x, th, n, heads, dtype, pad=pad), oracle.forward(x64, th, n, heads), dtype, tag + " fwd")
        gu.check_rotated(gu.run_transform(x, th, n, heads, dtype, inverse=True, pad=pad), oracle.inverse(x64, th, n, heads), dtype, tag + " inv")
    codes, scales = gu.run_fwd_quant(x, th, n, heads, dtype, 4, min(n, 128), "f16")
    gu.check_fused_codes(codes, scales, oracle.forward(x64, th, n, heads), 4, min(n, 128), "f16", dtype, tag)


@pytest.mark.parametrize("n,rows", [(256, 17), (1024, 5), (2048, 3)])
@pytest.mark.parametrize("dtype", ["f16", "f32"])
@pytest.mark.parametrize("bits,group,sd", [(4, 128, "f16"), (2, 64, "f32"), (4, 256, "f16")])
def test_short_last_block_stored_without_counts(n, rows, dtype, bits, group, sd):
    # fake-quantised rows alone (no bin counters): a variant of its own
    x, th, _ = synth.small_case(n, rows, dtype, seed=800 + n)
    codes, scales = gu.run_fwd_quant(x, th, n, 1, dtype, bits, group, sd)
    want = synth.cast_storage(oracle.dequantize(oracle.unpack_codes(codes, bits), scales.astype(np.float32), group).astype(np.float64), dtype)
    yq, _ = gu.run_fwd_fakequant(x, th, n, 1, dtype, bits, group, sd, want_hist=False)
    u = np.uint16 if dtype != "f32" else np.uint32
    np.testing.assert_array_equal(yq.view(u), want.view(u), err_msg=f"n={n} {dtype}")


@pytest.mark.parametrize("n,heads,rows,dtype", [
    (2048, 1, (1 << 16) + 1, "f16"), (256, 1, (1 << 19) + 5, "bf16"),  # 16-bit rows beyond the memory-side cache, one launch
    (1024, 2, (1 << 17) + 1, "bf16"), (256, 1, (1 << 20) + 5, "f16"),  # ... and the short block as a launch of its own
    (2048, 1, (1 << 15) + 1, "f32"), (512, 2, (1 << 16) + 3, "f32")])  # float32 rows: likewise for the codes
def test_large_batches_with_a_short_last_block(n, heads, rows, dtype):
    # rows at the front, in the middle and at the end (whole blocks and the short one) against the oracle; nothing behind the last
    # row or beside the rows is written; a row has the same bits in a short block as in a whole one
    import torch
    from paper_2509_09679_amd import binding as B

    dev, w = "cuda:0", n * heads
    rng = np.random.default_rng(900 + n)
    th = (rng.standard_normal((heads, n.bit_length() - 1, n // 2)) * 0.7).astype(np.float32)
    plan = B.alloc_plan(torch.from_numpy(th).to(dev), n, heads)
    gen = torch.Generator(device=dev).manual_seed(n)
    t = synth.torch_dtype(dtype)
    x = torch.empty((rows, w), dtype=t, device=dev)
    for r in range(0, rows, 1 << 14):
        x[r:r + (1 << 14)] = torch.randn(x[r:r + (1 << 14)].shape, generator=gen, device=dev).to(t)
    block = 4096 // w
    pick = torch.tensor([0, 1, block, rows // 2] + list(range(rows - 2 * block - 1, rows)), device=dev)
    end = x[rows - 2 * block:].contiguous()  # the last rows as whole blocks
    xs = synth.to_f64(synth.torch_to_storage(x[pick], dtype), dtype)
    store = lambda a: synth.torch_to_storage(a, dtype)
    tag = f"n={n} H={heads} T={rows} {dtype}"
    for inverse, ref in ((False, oracle.forward(xs, th, n, heads)), (True, oracle.inverse(xs, th, n, heads))):
        call = B.bq_butterfly_inv if inverse else B.bq_butterfly_fwd
        out = torch.full((rows + 3, w + 8), 7.0, dtype=t, device=dev)
        call(x, out, plan, B.make_rows(x, n, heads, out=out[:rows]))
        whole = torch.empty_like(end)
        call(end, whole, plan, B.make_rows(end, n, heads))
        gu.check_rotated(store(out[pick, :w].contiguous()), ref, dtype, f"{tag} inverse={inverse}")
        assert torch.equal(out[rows - 2 * block:rows, :w], whole)
        assert (out[rows:] == 7.0).all() and (out[:, w:] == 7.0).all()
        del out
    back = x.clone()
    B.bq_butterfly_fwd(back, back, plan, B.make_rows(back, n, heads))
    y = back[pick]
    B.bq_butterfly_inv(back, back, plan, B.make_rows(back, n, heads))
    gu.check_rotated(store(back[pick]), oracle.inverse(synth.to_f64(store(y), dtype), th, n, heads), dtype, tag + " in place")
    ref = oracle.forward(xs, th, n, heads)
    for bits, group, sd in ((2, 128, "f16"), (4, 64, "f32"), (4, 256, "f16")):
        q, spec = B.alloc_quant_outputs(rows + 1, n, heads, bits, group, sd, dev), B.make_quant(bits, group, sd)
        q[0][rows:], q[1][rows:] = 77, 7.0
        B.bq_butterfly_fwd_quant(x, plan, q[0], q[1], spec, B.make_rows(x, n, heads))
        whole = B.alloc_quant_outputs(2 * block, n, heads, bits, group, sd, dev)
        B.bq_butterfly_fwd_quant(end, plan, whole[0], whole[1], spec, B.make_rows(end, n, heads))
        gu.check_fused_codes(q[0][pick].cpu().numpy(), q[1][pick].cpu().numpy(), ref, bits, group, sd, dtype, tag)
        for a, b, guard in zip(q, whole, (77, 7.0)):
            assert torch.equal(a[rows - 2 * block:rows], b) and (a[rows:] == guard).all()


@pytest.mark.parametrize("n,heads,rows", [(4096, 1, 255), (4096, 1, 257), (4096, 1, 515), (8192, 1, 1), (8192, 1, 9), (8192, 1, 130),
                                          (2048, 2, 300), (512, 1, 70)])
def test_backward_at_the_slot_counts(n, heads, rows):
    # batches that fill no, some and several rows per slot; n = 8192 rounds the slots up to whole rounds of the dies, so some
    # of them have no rows and must still write their zeros
    x, th, dy = synth.small_case(n, rows, "f16", heads=heads, seed=700 + n + rows, with_dy=True, outliers=0)
    rdx, rdth, ab = oracle.backward(synth.to_f64(x, "f16"), synth.to_f64(dy, "f16"), th, n, heads)
    dx, dth = gu.run_bwd(x, dy, th, n, heads, "f16")
    gu.check_rotated(dx, rdx, "f16", f"dx n={n} T={rows}")
    floor = np.median(ab, axis=2, keepdims=True) if rows < 32 else ab  # (few rows: as in the seeded sweep)
    gu.check_dtheta(dth, rdth, np.maximum(ab, floor), what=f"dtheta n={n} T={rows}")


@pytest.mark.parametrize("n,heads,rows", [(512, 1, 3000), (512, 8, 300), (256, 1, 10), (2048, 1, 600), (8192, 1, 300), (4096, 1, 1501),
                                          (2048, 1, 2103), (1024, 2, 1101)])
def test_backward_of_flagged_plans_with_grown_tiles(n, heads, rows):
    # more tiles than workgroups: they grow, and their last one is ragged; fewer: workgroups without a slot take them
    x, th, dy = synth.small_case(n, rows, "f32", heads=heads, seed=800 + n + rows, with_dy=True, outliers=0)
    th = th.copy()
    th[:, :3] = np.float32(np.pi / 2)
    rdx, rdth, ab = oracle.backward(synth.to_f64(x, "f32"), synth.to_f64(dy, "f32"), th, n, heads)
    dx, dth = gu.run_bwd(x, dy, th, n, heads, "f32")
    gu.check_rotated(dx, rdx, "f32", f"dx n={n} T={rows}")
    floor = np.median(ab, axis=2, keepdims=True) if rows < 32 else ab
    gu.check_dtheta(dth, rdth, np.maximum(ab, floor), what=f"dtheta n={n} T={rows}")


@pytest.mark.parametrize("n,heads,rows", [(128, 1, 5), (128, 32, 3), (128, 32, 700), (64, 24, 40), (32, 3, 77), (8, 1, 600), (16, 4, 1)])
@pytest.mark.parametrize("dtype", ["f16", "f32"])
def test_small_quantisers_on_flagged_plans(n, heads, rows, dtype):
    # plain rotations held in registers; quantiser groups of the whole transform (their own instantiation) and smaller
    x, th, _ = synth.small_case(n, rows, dtype, heads=heads, seed=900 + n + rows)
    th = th.copy()
    th[:, :3] = np.float32(np.pi / 2)
    ref = oracle.forward(synth.to_f64(x, dtype), th, n, heads)
    for bits, group, sd in ((4, n, "f16"), (2, n, "f32"), (4, 8, "f32")):
        tag = f"n={n} H={heads} T={rows} {dtype} INT{bits} g{group} {sd}"
        codes, scales = gu.run_fwd_quant(x, th, n, heads, dtype, bits, group, sd)
        gu.check_fused_codes(codes, scales, ref, bits, group, sd, dtype, tag)
        c = oracle.unpack_codes(codes, bits)
        yq, hist = gu.run_fwd_fakequant(x, th, n, heads, dtype, bits, group, sd)
        want = synth.cast_storage(oracle.dequantize(c, scales.astype(np.float32), group).astype(np.float64), dtype)
        u = np.uint16 if dtype != "f32" else np.uint32
        np.testing.assert_array_equal(yq.view(u), want.view(u), err_msg=tag)
        np.testing.assert_array_equal(hist, oracle.bin_histogram(c, bits), err_msg=tag)


@pytest.mark.parametrize("op", ["fwd", "inv", "quant", "fake"])
def test_small_transforms_of_rows_far_apart(op):
    # A workgroup takes four rows of 128 or more at a time and a lane's offset among them has 32 bits; rows 1.5 GB apart must be groups
    # of their own.  Row 3 lies 4.5 GB behind row 0: an offset of 32 bits would come out 0.5 GB behind it, where nothing is a row's
    # (all wrapped places hold 7, so a load from one shows in the result and a store to one in what it holds).
    import torch
    from paper_2509_09679_amd import binding as B

    n, ld = 128, (3 << 28) + 256
    rows = 4 if op in ("fwd", "inv") else 16
    starts = [r * ld for r in range(rows)]
    wrapped = [s % (1 << 31) for s in starts if 2 * s >= 1 << 32]  # in elements of two bytes
    assert wrapped and not set(wrapped) & set(starts)
    x, th, _ = synth.small_case(n, rows, "f16", seed=11)
    plan = B.alloc_plan(torch.from_numpy(th).cuda(), n, 1)
    dense = torch.from_numpy(np.ascontiguousarray(x).view(np.float16)).cuda()

    def far(fill):
        buf = torch.empty((rows - 1) * ld + n, dtype=torch.float16, device="cuda")
        for w in wrapped:
            buf[w:w + n] = 7.0
        view = buf.as_strided((rows, n), (ld, 1))
        view.copy_(fill)
        return buf, view

    if op in ("fwd", "inv"):
        f = B.bq_butterfly_fwd if op == "fwd" else B.bq_butterfly_inv
        call = lambda a, b: f(a, b, plan, B.make_rows(a, n, 1, out=b))  # noqa: E731
    elif op == "fake":
        q = B.make_quant(4, 32, "f16")
        call = lambda a, b: B.bq_butterfly_fwd_fakequant(a, plan, b, None, q, B.make_rows(a, n, 1, out=b))  # noqa: E731
    if op != "quant":
        want = torch.empty_like(dense)
        call(dense, want)
        xs, got = far(dense)[1], torch.empty_like(dense)
        call(xs, got)  # loads far apart
        assert torch.equal(got, want)
        del xs
        buf, ys = far(torch.zeros_like(dense))
        call(dense, ys)  # stores far apart
        assert torch.equal(ys, want) and all(bool((buf[w:w + n] == 7.0).all()) for w in wrapped)
        return
    codes, scales = B.alloc_quant_outputs(rows, n, 1, 4, 32, "f32", "cuda")
    codes2, scales2 = torch.zeros_like(codes), torch.zeros_like(scales)
    q = B.make_quant(4, 32, "f32")
    B.bq_butterfly_fwd_quant(dense, plan, codes, scales, q, B.make_rows(dense, n, 1))
    xs = far(dense)[1]
    B.bq_butterfly_fwd_quant(xs, plan, codes2, scales2, q, B.make_rows(xs, n, 1))
    assert torch.equal(codes, codes2) and torch.equal(scales, scales2)


@pytest.mark.parametrize("n,heads,rows", [(4096, 1, 3), (4096, 1, 1303), (4096, 3, 171), (1024, 1, 1301), (8192, 1, 130)])
@pytest.mark.parametrize("dtype", ["f32", "f16", "bf16"])
def test_large_groups_with_either_scale_type(n, heads, rows, dtype):
    # kernels with the scale types apart and together; how a workgroup's bin counts are added up at its end differs by what is stored, row
    # type and size; every sixteenth row is so small that its binary16 scale is subnormal and the clip acts
    x, th, _ = synth.small_case(n, rows, "f32", heads=heads, seed=950 + n + rows)
    x[::16] *= np.float32(1e-6 / np.abs(x[::16]).max())
    x = synth.cast_storage(x.astype(np.float64), dtype)
    ref = oracle.forward(synth.to_f64(x, dtype), th, n, heads)
    ordinary = np.arange(rows) % 16 != 0
    u = np.uint16 if dtype != "f32" else np.uint32
    for bits, group, sd in ((2, 256, "f16"), (2, n, "f32"), (4, n, "f16"), (4, 256, "f32")):
        tag = f"n={n} H={heads} T={rows} {dtype} INT{bits} g{group} {sd}"
        codes, scales = gu.run_fwd_quant(x, th, n, heads, dtype, bits, group, sd)
        gu.check_fused_codes(codes[ordinary], scales[ordinary], ref[ordinary], bits, group, sd, dtype, tag)
        c = oracle.unpack_codes(codes, bits)
        want = synth.cast_storage(oracle.dequantize(c, scales.astype(np.float32), group).astype(np.float64), dtype)
        for want_y, want_hist in ((True, True), (True, False), (False, True)):
            yq, hist = gu.run_fwd_fakequant(x, th, n, heads, dtype, bits, group, sd, want_y=want_y, want_hist=want_hist)
            if want_y:
                np.testing.assert_array_equal(yq.view(u), want.view(u), err_msg=tag)
            if want_hist:
                np.testing.assert_array_equal(hist, oracle.bin_histogram(c, bits), err_msg=tag)
