"""Checks of the host side of libpatconv.so that need no GPU: every HIP call goes to tests/_hip_stub.c, so the launches of a call can be
looked at. Runs as a program of its own (the stub has to be loaded before any HIP library): python -m tests._host_probe STUB CHECK."""
import ctypes as ct
import struct
import sys
import time

stub = ct.CDLL(sys.argv[1], ct.RTLD_GLOBAL)

from paper_2011_10170_amd import binding as B  # noqa: E402
from paper_2011_10170_amd import inputs as I  # noqa: E402

LIB = I.make_library(8)
DEV = 1 << 20        # stands for a device address; nothing reads it


def watch(name, arg=0, nbytes=0):
    """The launches of kernels with `name` in their symbol are noted from here on, with the first bytes of one of their arguments."""
    ct.memmove(ct.addressof(ct.c_char.in_dll(stub, "stub_watch")), name.encode() + b"\0", len(name) + 1)
    ct.c_int.in_dll(stub, "stub_arg").value = arg
    ct.c_int.in_dll(stub, "stub_arg_bytes").value = nbytes


def seen():
    n = ct.c_int.in_dll(stub, "stub_arg_bytes").value
    return (ct.string_at(ct.addressof(ct.c_char.in_dll(stub, "stub_args")), n), ct.c_longlong.in_dll(stub, "stub_grid").value,
            ct.c_longlong.in_dll(stub, "stub_lds").value)


def layer(ctx, shape, read=True, keep=0.3):
    """Descriptor and pack of a layer; read: its kept-kernel count is known on the host, as after a read-back."""
    N, H, W, C, F, st = shape
    pk = B.pc_pack(ctx, DEV, DEV, DEV, F, C, LIB, B.PC_BF16)
    ct.c_int.in_dll(stub, "stub_count").value = F * I.kept_per_filter(keep, C)
    if read:
        B.pc_packed_info(ctx, pk)
    return B.make_desc(N, H, W, C, F, st, B.PC_BF16), pk


def wgrad_lds():
    """Backward-weight with direct loads: every column that a wavefront reads ahead lies inside the workgroup's LDS."""
    ctx = B.pc_create(0, None)
    B.pc_set_plan_override(ctx, 44, 0)
    tiles = set()
    for st in (1, 2):
        for N in (1, 3, 9, 70):
            for H in (1, 2, 4, 7, 16, 33):
                for W in (1, 2, 3, 4, 5, 6, 7, 8, 9, 14, 47):
                    d, pk = layer(ctx, (N, H, W, 64, 64, st))
                    watch("pc_mfma_wgrad_dma_kernel", 0, 88 + 64)
                    B.pc_conv_bwd_weight(ctx, d, pk, DEV, DEV, DEV)
                    arg, _, lds = seen()
                    TR, TC, IW, nrow, RPx, RPd, dy_off = struct.unpack("<16i", arg[88:])[9:]
                    tiles.add((st, TC))
                    # the last column of dy and of x that is asked for, and the bytes of the last staged row up to its end
                    d_col = min(7, IW) if st == 1 else max([c + 3 for c in (0, 2) if c < TC] + [TC - 1])
                    x_col = min(9, IW) if st == 1 else max(c + 2 for u in range(8) for c in [4 * (u // 3) + (u % 3 + 1 if u % 3 < 2 else 4)] if 2 * (u // 3) < TC)
                    assert dy_off + (TR - 1) * RPd + (d_col + 1) * 128 <= lds <= 80 * 1024, (N, H, W, st, TR, TC, lds)
                    assert (nrow - 1) * RPx + (x_col + 1) * 128 <= lds and nrow * RPx <= dy_off, (N, H, W, st, TR, TC, lds)
                    B.pc_packed_free(pk)
    assert len(tiles) >= 9, tiles
    B.pc_destroy(ctx)


def wgrad_lds_narrow():
    """The same where wavefronts share the pixels of a tile (split_k 1 to 3): every wavefront's columns, and the sums they add in LDS."""
    ctx = B.pc_create(0, None)
    tiles = set()
    for waves, (fw, cw) in ((1, (1, 2)), (2, (2, 1)), (3, (1, 1))):
        B.pc_set_plan_override(ctx, 44, waves)
        for st in (1, 2):
            for N in (1, 9, 70):
                for H in (1, 4, 7, 33, 200):
                    for W in (1, 2, 3, 5, 8, 14, 47, 190):
                        d, pk = layer(ctx, (N, H, W, 24, 40, st))
                        watch("pc_mfma_wgrad_dma_kernel", 0, 88 + 112)
                        B.pc_conv_bwd_weight(ctx, d, pk, DEV, DEV, DEV)
                        arg, grid, lds = seen()
                        a = struct.unpack("<28i", arg[88:])
                        TR, TC, IW, nrow, RPx, RPd, dy_off = a[9:16]
                        assert a[25] == waves and a[18] >= 1 and grid == -(-24 // (32 * cw)) * -(-40 // (32 * fw)) * a[18]
                        lgPC, NC, XB, DB = a[26], a[27], 64 * cw, 64 * fw
                        tiles.add((st, waves, lgPC, TR, NC))
                        assert 4 * 18 * 1024 <= lds <= 80 * 1024 and nrow * RPx <= dy_off and TC * DB <= min(1024, RPd) and IW * XB <= min(2048, RPx)
                        assert TR % (((32 if st == 1 else 16) * 4 // (fw * cw)) >> lgPC) == 0
                        for p in range(1 << lgPC):
                            nc = min(NC, TC - p * NC)
                            if nc <= 0:
                                continue
                            d_col = p * NC + (min(7, nc + 2) if st == 1 else max([c + 3 for c in (0, 2) if c < nc] + [nc - 1]))
                            x_col = p * NC * st + (min(9, nc + 2) if st == 1 else
                                                   max(c + 2 for u in range(8) for c in [4 * (u // 3) + (u % 3 + 1 if u % 3 < 2 else 4)] if 2 * (u // 3) < nc))
                            assert dy_off + (TR - 1) * RPd + (d_col + 1) * DB <= lds, (N, H, W, st, waves, a)
                            assert (nrow - 1) * RPx + (x_col + 1) * XB <= lds, (N, H, W, st, waves, a)
                        B.pc_packed_free(pk)
    assert len(tiles) >= 30, len(tiles)
    B.pc_destroy(ctx)


def alignment():
    """Tensors whose address is no multiple of 16 go to the kernels that load through registers, before and after an aligned call of the
    same sizes, and back."""
    ctx = B.pc_create(0, None)
    direct = 0
    kernels = ("conv_dma", "conv_solo", "conv_ring", "conv_keep", "conv_deep", "wgrad_dma_few", "wgrad_dma")
    met = set()
    for shape in [(9, 38, 41, 56, 64, 1), (32, 112, 112, 128, 128, 1), (64, 7, 7, 512, 512, 1), (64, 56, 56, 128, 128, 2), (64, 14, 14, 256, 512, 2), (13, 33, 47, 40, 72, 1),
                  (32, 224, 224, 64, 64, 1), (61, 199, 198, 32, 16, 1), (1, 14, 14, 512, 512, 1), (128, 2, 2, 256, 512, 1)]:
        d, pk = layer(ctx, shape)
        calls = [lambda a: B.pc_conv_fwd(ctx, d, pk, a, DEV), lambda a: B.pc_conv_bwd_data(ctx, d, pk, a, DEV), lambda a: B.pc_conv_bwd_data_relu(ctx, d, pk, a, DEV, DEV),
                 lambda a: B.pc_conv_bwd_weight(ctx, d, pk, a, DEV, DEV), lambda a: B.pc_conv_bwd_weight(ctx, d, pk, DEV, a, DEV),
                 lambda a: B.pc_conv_bwd_weight_batch(ctx, [d], [pk], [a], [DEV], [DEV]), lambda a: B.pc_conv_bwd_weight_batch(ctx, [d], [pk], [DEV], [a], [DEV])]
        for call in calls:
            names = []
            for off in (2, 0, 8, 0):
                call(DEV + off)
                names.append(B.pc_last_kernel(ctx))
            is_direct = [any(k in n for k in kernels) for n in names]
            met.update(k for k in kernels if any(k in n for n in names))
            assert not is_direct[0] and not is_direct[2] and names[0] == names[2] and names[1] == names[3], (shape, names)
            direct += is_direct[1]
        small = shape[0] * shape[1] * shape[2] < 4096
        for code in (41, 43, 44) + ((50,) if max(shape[3:5]) <= 64 else ()) + ((51, 53, 55) if small else ()) if shape[5] == 1 else (44, 48):      # forced, they are refused
            B.pc_set_plan_override(ctx, code, 0)
            call = calls[3] if code in (44, 55) else calls[0]
            call(DEV)
            try:
                call(DEV + 4)
                assert False, (shape, code)
            except B.PcError as e:
                assert e.status == B.PC_ERR_UNSUPPORTED
            B.pc_set_plan_override(ctx, -1, 0)
        B.pc_packed_free(pk)
    assert direct >= 40 and met == set(kernels), (direct, met)
    B.pc_destroy(ctx)


def thin_planes():
    """The first layer's weight gradient: about two workgroups per CU however many filters there are, and partial planes within 32 MiB."""
    ctx = B.pc_create(0, None)
    for st in (1, 2):
        for N, H, W in ((1, 1, 2), (3, 33, 47), (32, 224, 224)):
            for C, F in ((3, 8), (3, 64), (4, 72), (3, 512), (4, 1024), (3, 2048), (4, 65528)):
                if N * H * W * F >= 1 << 30:
                    continue
                d, pk = layer(ctx, (N, H, W, C, F, st), read=False)
                watch("pc_thin_wgrad_kernel")
                B.pc_conv_bwd_weight(ctx, d, pk, DEV, DEV, DEV)
                assert B.pc_last_kernel(ctx).startswith("pc_thin_wgrad_kernel")
                grid, blocks = seen()[1], (F + 63) // 64
                splits = grid // blocks
                assert splits * blocks == grid and splits >= 1 and (splits == 1 or grid <= 2 * 256), (N, H, W, C, F, st, grid)
                assert splits == 1 or splits * F * C * 16 <= 32 << 20, (N, H, W, C, F, st, grid)
                B.pc_packed_free(pk)
    B.pc_destroy(ctx)


def noalloc_first_layer():
    """The entry point that allocates nothing: the kernel of the call that does, or a refusal where the partial planes of the wave-specialised
    kernel and the 8-channel copy of x that it reads exceed 32 MiB."""
    ctx = B.pc_create(0, None)
    for shape, fits in (((32, 208, 208, 3, 512, 1), True), ((40, 224, 224, 3, 64, 1), True), ((43, 224, 224, 3, 64, 1), False), ((43, 224, 224, 4, 128, 1), False),
                        ((8, 64, 64, 3, 512, 1), True), ((32, 208, 208, 1, 2048, 2), True), ((128, 32, 32, 3, 64, 1), True)):
        for read in (True, False):
            d, pk = layer(ctx, shape, read=read)
            B.pc_conv_bwd_weight(ctx, d, pk, DEV, DEV, DEV)
            want = B.pc_last_kernel(ctx)
            watch("wgrad", 0, 0)
            ct.c_longlong.in_dll(stub, "stub_grid").value = 0
            try:
                B.pc_conv_bwd_weight_noalloc(ctx, d, pk, DEV, DEV, DEV)
                assert fits and B.pc_last_kernel(ctx) == want and want.startswith("pc_thin_wgrad_kernel"), (shape, want, B.pc_last_kernel(ctx))
            except B.PcError as e:
                assert not fits and e.status == B.PC_ERR_UNSUPPORTED and seen()[1] == 0, (shape, e)
            B.pc_packed_free(pk)
    B.pc_destroy(ctx)


def no_host_memory():
    """No C++ exception leaves a C entry or the binding: an allocation on the host that fails, whichever it is, is an error of the call."""
    ctx = B.pc_create(0, None)
    ls = [layer(ctx, s) for s in [(8, 32, 32, 3, 64, 1), (8, 32, 32, 64, 64, 1), (8, 16, 16, 64, 128, 1), (8, 16, 16, 12, 20, 1)]]
    n = [DEV] * len(ls)
    hist = (ct.c_uint32 * 512)(*range(512))
    left = ct.c_int.in_dll(stub, "stub_new_left")
    for name, call in (("batch", lambda: B.pc_conv_bwd_weight_batch(ctx, [d for d, _ in ls], [p for _, p in ls], n, n, [DEV + 64 * i for i in range(len(ls))])),
                       ("fallback", lambda: B.pc_conv_bwd_weight_batch(ctx, [d for d, _ in ls[1:]], [p for _, p in ls[1:]], n[1:], n[1:], [DEV + 64 * i for i in range(1, len(ls))])),
                       ("one", lambda: B.pc_conv_bwd_weight(ctx, *ls[0], DEV, DEV, DEV)), ("pool", lambda: B.pc_dppg_pool(ctx, ct.addressof(hist), 8))):
        for k in range(1, 1000):
            left.value = k
            try:
                call()
                if left.value > 0:          # fewer allocations than k
                    left.value = 0
                    break
            except MemoryError:
                left.value = 0
            except B.PcError as e:
                left.value = 0
                assert e.status == B.PC_ERR_NOMEM, (name, k, e)
        print(name, k)
        assert k < 999 and (k > 10) == (name in ("batch", "fallback"))
        call()
    for _, p in ls:
        B.pc_packed_free(p)
    B.pc_destroy(ctx)


def no_room():
    """Backward-weight where the scratch buffer cannot grow: another kernel takes the call, which succeeds and leaves no message. The entry
    point that allocates nothing goes to the kernel of the call that has room."""
    for dims in ([(32, 28, 28, 512, 512, 1)], [(32, 112, 112, 128, 128, 1), (32, 56, 56, 256, 256, 1), (32, 28, 28, 512, 512, 1)]):
        ctx = B.pc_create(0, None)
        ls = [layer(ctx, s) for s in dims]
        n = [DEV] * len(ls)

        def call(noalloc=False):
            if noalloc:
                B.pc_conv_bwd_weight_noalloc(ctx, *ls[0], DEV, DEV, DEV)
            elif len(ls) == 1:
                B.pc_conv_bwd_weight(ctx, *ls[0], DEV, DEV, DEV)
            else:
                B.pc_conv_bwd_weight_batch(ctx, [d for d, _ in ls], [p for _, p in ls], n, n, [DEV + 64 * i for i in range(len(ls))])
            return B.pc_last_kernel(ctx)

        B.pc_set_plan_override(ctx, 11, 0)
        assert "wgrad_ws" in call()
        B.pc_set_plan_override(ctx, -1, 0)
        for name in ("stub_malloc_fails", "stub_capturing"):
            ct.c_int.in_dll(stub, name).value = 1
            assert "wgrad_ws" in call()
            assert B.load().pc_last_error(ctx) == b"", B.load().pc_last_error(ctx)
            if len(ls) == 1:
                assert "wgrad_dma" in call(noalloc=True)
            ct.c_int.in_dll(stub, name).value = 0
        assert "wgrad_dma" in call()
        ct.c_int.in_dll(stub, "stub_capturing").value = 1
        assert "wgrad_dma" in call()
        ct.c_int.in_dll(stub, "stub_capturing").value = 0
        for _, p in ls:
            B.pc_packed_free(p)
        B.pc_destroy(ctx)


def no_room_first_layer():
    """The same for first layers, alone and beside other layers: their partial planes, too, make way for the kernel that needs less."""
    for dims in ([(8, 64, 64, 3, 512, 1)], [(8, 64, 64, 3, 512, 1), (8, 64, 64, 64, 64, 1)], [(4, 64, 64, 4, 1024, 1)], [(8, 64, 64, 64, 64, 1), (2, 33, 9, 3, 2048, 2), (5, 40, 41, 3, 64, 1)]):
        for read in (True, False):
            ctx = B.pc_create(0, None)
            ls = [layer(ctx, s, read=read) for s in dims]
            n = [DEV] * len(ls)

            def call():
                B.pc_conv_bwd_weight_batch(ctx, [d for d, _ in ls], [p for _, p in ls], n, n, [DEV + 64 * i for i in range(len(ls))])
                return B.pc_last_kernel(ctx)

            B.pc_set_plan_override(ctx, 11, 0)
            assert "wgrad_ws" in call()
            B.pc_set_plan_override(ctx, -1, 0)
            for name in ("stub_malloc_fails", "stub_capturing"):
                ct.c_int.in_dll(stub, name).value = 1
                kernel = call()
                assert "wgrad" in kernel and B.load().pc_last_error(ctx) == b"", (dims, kernel)
                ct.c_int.in_dll(stub, name).value = 0
            assert "wgrad_dma" in call() or "thin_wgrad" in B.pc_last_kernel(ctx)
            for _, p in ls:
                B.pc_packed_free(p)
            B.pc_destroy(ctx)


def changing_counts():
    """A layer whose kept count differs after every re-pack is not planned again in every call: such calls cost about what calls of one count do."""
    ctx = B.pc_create(0, None)
    for dtype in (B.PC_F32, B.PC_BF16):
        for N, H, W, C, F, st in ((64, 28, 28, 128, 128, 1), (13, 33, 47, 40, 72, 1), (32, 64, 64, 3, 64, 1)):
            d, pk = B.make_desc(N, H, W, C, F, st, dtype), B.pc_pack(ctx, DEV, DEV, DEV, F, C, LIB, dtype)

            def median(counts):
                us = []
                for n in counts:
                    ct.c_int.in_dll(stub, "stub_count").value = n
                    B.pc_pack(ctx, DEV, DEV, DEV, F, C, LIB, dtype, reuse=pk)
                    B.pc_packed_info(ctx, pk)
                    t = time.perf_counter()
                    B.pc_conv_bwd_weight(ctx, d, pk, DEV, DEV, DEV)
                    us.append((time.perf_counter() - t) * 1e6)
                return sorted(us)[len(us) // 2]

            n0 = F * C * 5 // 16
            same, new = median([n0] * 101), median([n0 - i for i in range(1, 102)])
            print((dtype, N, H, W, C, F), "%.1f %.1f us" % (same, new))
            assert new <= 2.0 * same + 2.0, (dtype, N, H, W, C, F, same, new)
            B.pc_packed_free(pk)
    B.pc_destroy(ctx)


def kernel_code(name):
    """The override code of a forward / backward-data kernel by its symbol."""
    v = name.split("<")[1].rstrip(">").split(", ")
    if "conv_ks" in name:
        return {"2 4 4 64": 7, "2 2 4 64": 8, "2 1 4 64": 9, "2 1 4 128": 14, "1 1 4 128": 15, "2 2 1 32": 16, "2 4 1 16": 17, "2 2 1 16": 18, "1 4 1 32": 19, "2 2 1 64": 20,
                "2 2 4 128": 21, "1 2 1 64": 24, "1 2 1 32": 25, "1 4 1 16": 26, "1 2 4 128": 27, "1 4 4 64": 28, "1 2 4 64": 29, "2 2 2 32": 30, "2 4 2 16": 31}[" ".join((v[0], v[1], v[4], v[3]))]
    if "conv_dma" in name:
        return {"8": 40, "4": 41, "7": 42}[v[0]]
    if "conv_solo" in name:
        return {"0 2 4": 43, "0 4 4": 45, "0 2 2": 46, "1 2 4": 47, "1 2 2": 48, "2 2 4": 37, "2 2 2": 38}[" ".join(v[:3])]
    if "conv_mc" in name:
        return {"2 64": 32, "2 32": 33, "2 16": 34, "1 64": 35, "1 32": 36}[" ".join(v[:2])]
    if "conv_ring" in name:
        return 49
    if "conv_keep" in name:
        return 50
    if "conv_deep" in name:
        return {"1 2": 51, "1 4": 52, "2 2": 53, "2 4": 54}[" ".join(v[:2])]
    return {"2 4 2 2 32": 1, "2 2 2 2 64": 3, "1 2 2 2 64": 4, "1 1 2 2 64": 5, "1 2 2 2 16": 6}[" ".join(v[:4] + v[5:6])]


def conv_choice():
    """The kernel that a forward or backward-data pass goes to against the stored timings of every kernel that takes it; layers of 8 and 16 input
    channels, where the cooperative kernel (6) is among them, by themselves. Unaligned tensors: against the kernels without direct loads."""
    times = {}
    for row in open("profiles/plan_timings_bf16.csv"):
        f = row.strip().split(",")
        if f[0] in ("fwd", "bwd_data"):
            times.setdefault((f[0],) + tuple(int(v) for v in f[1:7]), {})[int(f[7])] = float(f[8])
    ctx = B.pc_create(0, None)
    for off in (0, 2):
        late = {}
        for k, us in times.items():
            d, pk = layer(ctx, k[1:])
            (B.pc_conv_fwd if k[0] == "fwd" else B.pc_conv_bwd_data)(ctx, d, pk, DEV + off, DEV)
            code = kernel_code(B.pc_last_kernel(ctx))
            best = min(v for c, v in us.items() if not off or not 37 <= c <= 54)
            if code in us:      # (what was timed of a layer leaves out kernels that are never near)
                late.setdefault((k[0], k[6], (k[4] if k[0] == "fwd" else k[5]) <= 16), []).append(us[code] / best)
            B.pc_packed_free(pk)
        assert sum(len(v) for v in late.values()) >= 0.95 * len(times)
        for k, v in late.items():
            print(off, k, len(v), sum(v) / len(v), max(v))
            assert len(v) < 10 or (sum(v) / len(v) < (1.025 if off == 0 else 1.05) and max(v) < (1.25 if off == 0 else 1.5)), (off, k)
    B.pc_destroy(ctx)


def stored(path, n_key, n_plan, words=0):
    """{what the plan is made for: {plan: us}} of a file of stored timings; words: leading columns that are no numbers."""
    times = {}
    for row in list(open(path))[1:]:
        f = row.strip().split(",")
        v = tuple(f[:words]) + tuple(int(x) for x in f[words:-1])
        times.setdefault(v[:n_key], {})[v[n_key:n_key + n_plan]] = float(f[-1])
    return times


def compare(what, late, mean, worst, missing):
    """late: the chosen plan's stored time over the least one of each layer, None where that plan was not timed. Bounds: what these layers
    show, and as much again as two runs of a time differ by (2 % in the mean, 5 % of one layer)."""
    got = [v for v in late if v is not None]
    print(what, len(late), len(late) - len(got), sum(got) / len(got), max(got))
    assert len(late) - len(got) <= missing * len(late) and sum(got) / len(got) < mean and max(got) < worst, what


def wgrad_choice():
    """A layer's weight gradient goes to the kernel with direct loads, and its arrangement of the wavefronts, pixel tile and splits are held against the
    stored times of those and others."""
    ctx = B.pc_create(0, None)
    late = []
    few = few_timings()
    for k, us in stored("profiles/wgrad_plan_timings_bf16.csv", 6, 5).items():
        d, pk = layer(ctx, k)
        watch("pc_mfma_wgrad_dma_kernel", 0, 88 + 112)
        B.pc_conv_bwd_weight(ctx, d, pk, DEV, DEV, DEV)
        assert "wgrad_dma" in B.pc_last_kernel(ctx), k
        if "wgrad_dma_few" in B.pc_last_kernel(ctx):      # (another kernel: its stored times are looked at below)
            assert k in few, k
            B.pc_packed_free(pk)
            continue
        a = struct.unpack("<28i", seen()[0][88:])
        plan = (a[25], a[26], a[9], a[27], a[18])
        late.append(us[plan] / min(us.values()) if plan in us else None)
        B.pc_packed_free(pk)
    compare("bwd_weight", late, 1.057, 1.24, 0.05)      # 1.037, 1.19
    B.pc_destroy(ctx)


def few_timings():
    """{layer: {(code, tile): (us in a graph, us launch by launch)}} of the kernel for few pixels (55) and the one with direct loads (44)."""
    times = {}
    for row in list(open("profiles/wgrad_few_timings_bf16.csv"))[1:]:
        f = row.strip().split(",")
        times.setdefault(tuple(int(v) for v in f[:6]), {})[(int(f[6]), int(f[7]))] = (float(f[8]), float(f[9]))
    return times


def wgrad_few_choice():
    """Weight gradients of 4 to 8400 pixels: the kernel for few pixels or the one with direct loads, and the tile of either, against the stored times
    of all tiles of both: those in a graph, which the line between the two is drawn for, and those launch by launch."""
    ctx = B.pc_create(0, None)
    late, chosen = [], set()
    for k, us in few_timings().items():
        d, pk = layer(ctx, k)
        watch("pc_mfma_wgrad_dma_kernel", 0, 88 + 112)
        B.pc_conv_bwd_weight(ctx, d, pk, DEV, DEV, DEV)
        name = B.pc_last_kernel(ctx)
        if "wgrad_dma_few" in name:
            plan = (55, {"1, 1": 0, "1, 2": 1, "2, 1": 2, "2, 2": 3}[name.split("<")[1][:-1]])
        else:
            plan = (44, struct.unpack("<28i", seen()[0][88:])[25])
        chosen.add(plan)
        late.append([us[plan][i] / min(v[i] for v in us.values()) for i in range(2)])
        B.pc_packed_free(pk)
    assert {(55, 0), (55, 2), (55, 3), (44, 0), (44, 3)} <= chosen, chosen
    compare("in a graph", [v[0] for v in late], 1.032, 1.19, 0.0)              # 1.012, 1.14
    compare("launch by launch", [v[1] for v in late], 1.038, 1.31, 0.0)        # 1.018, 1.26
    B.pc_destroy(ctx)


def f32_wgrad_choice():
    """The same for float32 layers, those with few input channels by themselves."""
    ctx = B.pc_create(0, None)
    late = {}
    for k, us in stored("profiles/wgrad_plan_timings_f32.csv", 6, 5).items():
        N, H, W, C, F, st = k
        pk = B.pc_pack(ctx, DEV, DEV, DEV, F, C, LIB, B.PC_F32)
        ct.c_int.in_dll(stub, "stub_count").value = F * I.kept_per_filter(0.3, C)
        B.pc_packed_info(ctx, pk)
        watch("pc_f32_wgrad_kernel", 2, 17 * 4)
        B.pc_conv_bwd_weight(ctx, B.make_desc(N, H, W, C, F, st, B.PC_F32), pk, DEV, DEV, DEV)
        a = struct.unpack("<17i", seen()[0])
        plan = tuple(int(v) for v in B.pc_last_kernel(ctx).split("<")[1].split(",")[:2]) + (a[8], a[9], a[16])
        late.setdefault(C <= 3, []).append(us[plan] / min(us.values()) if plan in us else None)
        B.pc_packed_free(pk)
    compare("bwd_weight", late[False], 1.053, 1.2, 0.05)            # 1.033, 1.15
    compare("few channels", late[True], 1.117, 1.29, 0.05)          # 1.097, 1.24
    B.pc_destroy(ctx)


def f32_conv_choice():
    """The shape and chunk length of float32 forward and backward-data passes against the stored times of all that take the layer."""
    ctx = B.pc_create(0, None)
    late = {}
    times = {}
    for row in list(open("profiles/plan_timings_f32.csv"))[1:]:
        f = row.strip().split(",")
        times.setdefault((f[0],) + tuple(int(v) for v in f[1:7]), {})[f[7]] = float(f[8])
    for k, us in times.items():
        N, H, W, C, F, st = k[1:]
        pk = B.pc_pack(ctx, DEV, DEV, DEV, F, C, LIB, B.PC_F32)
        watch("pc_f32_conv_kernel", 3, 12 * 4)
        (B.pc_conv_fwd if k[0] == "fwd" else B.pc_conv_bwd_data)(ctx, B.make_desc(N, H, W, C, F, st, B.PC_F32), pk, DEV, DEV)
        plan = "x".join(B.pc_last_kernel(ctx).split("<")[1].split(", ")[:5]) + "/%d" % struct.unpack("<12i", seen()[0])[11]
        late.setdefault((k[0], st), []).append(us.get(plan, 1e9) / min(us.values()))
        B.pc_packed_free(pk)
    for k, v in late.items():                                        # 1.021 and 1.029, 1.25; stride 2 1.027 and 1.041, 1.18
        compare(k, v, 1.049 if k[1] == 1 else 1.061, 1.3, 0.0)
    B.pc_destroy(ctx)


def network(kind, width, images, size, stages):
    """The 3x3 layers of a VGG- or ResNet-shaped network (basic and bottleneck blocks)."""
    out, c = [], 3 if kind == "vgg" else width
    for s in range(stages):
        f = width * min(8, 1 << s)
        for k in range((2 if s < 2 else 3) if kind == "vgg" else 4 if kind == "basic" else (3, 4, 6, 3)[s]):
            st = 2 if kind != "vgg" and s and k == 0 else 1
            out.append((images, size, size, f if kind == "bottleneck" else c, f, st))
            size, c = (size - 1) // st + 1, f
        if kind == "vgg":
            size //= 2
    return out


def group_choice():
    """The weight gradients of a network in one call go to the kernel with direct loads, and the share of a workgroup (told by how many there are)
    is held against the stored times of eight."""
    times = {}
    for row in list(open("profiles/group_share_timings_bf16.csv"))[1:]:
        f = row.strip().split(",")
        times.setdefault(tuple(f[:7]), {})[int(f[8])] = float(f[9])
    ctx = B.pc_create(0, None)
    late = []
    for k, us in times.items():
        ls = [layer(ctx, s, read=k[6] == "yes", keep=float(k[5])) for s in network(k[0], *(int(v) for v in k[1:5]))]
        n = [DEV] * len(ls)
        watch("pc_mfma_wgrad_dma_group_kernel")
        B.pc_conv_bwd_weight_batch(ctx, [d for d, _ in ls], [p for _, p in ls], n, n, [DEV + 64 * i for i in range(len(ls))])
        assert "wgrad_dma_group" in B.pc_last_kernel(ctx), k
        late.append(us[seen()[1]] / min(us.values()) if seen()[1] in us else None)
        for _, p in ls:
            B.pc_packed_free(p)
    compare("group", late, 1.044, 1.29, 0.05)           # 1.024, 1.24
    B.pc_destroy(ctx)


if __name__ == "__main__":
    globals()[sys.argv[2]]()
    print("ok")
