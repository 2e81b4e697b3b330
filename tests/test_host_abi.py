"""Host side of the C ABI (no GPU): exported symbols, packer bytes vs the oracle, error codes."""
import ctypes as C
import os
import re

import numpy as np
import pytest
from hypothesis import given, settings, strategies as st

import paper_2602_01027_amd as S
from oracle import sfmp_oracle as O
import sfmp_workloads as W

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_library_exports_every_declared_symbol():
    header = open(os.path.join(ROOT, "include", "sfmp.h")).read()
    header = re.sub(r"/\*.*?\*/", "", header, flags=re.S)
    declared = set(re.findall(r"\b(sfmp_[a-z_0-9]+)\s*\(", header))
    assert declared == set(S.binding.EXPORTS), declared ^ set(S.binding.EXPORTS)
    lib = S.load_library()
    for name in declared:
        assert getattr(lib, name) is not None


def test_layout_struct_matches_header_size():
    # 8 int32 + 4 int64 + 2 int32 = 72 bytes, no padding
    assert C.sizeof(S.SfmpLayout) == 72


@settings(max_examples=10, deadline=None)
@given(st.integers(0, 2 ** 31 - 1), st.integers(1, 3), st.integers(1, 4))
def test_packer_bytes_equal_oracle(seed, ntr, ntc):
    rng = np.random.default_rng(seed)
    bitmap = rng.integers(2, 5, size=(ntr, ntc)).astype(np.int8)
    bm = np.repeat(np.repeat(bitmap, 128, axis=0), 128, axis=1)
    codes = (rng.integers(0, 16, size=bm.shape) % (1 << bm)).astype(np.uint8)
    L, s2, s3, s4, index = S.sfmp_pack(codes, bitmap)
    ref = O.pack(codes, bitmap)
    assert np.array_equal(s2, ref["s2"]) and np.array_equal(s3, ref["s3"]) and np.array_equal(s4, ref["s4"])
    assert np.array_equal(index, ref["index"])
    assert (L.N, L.K, L.tile, L.group) == (ntr * 128, ntc * 128, 128, 128)
    assert (L.count2, L.count3, L.count4) == tuple(int((bitmap == b).sum()) for b in (2, 3, 4))
    assert (L.bytes_s2, L.bytes_s3, L.bytes_s4) == (s2.size, s3.size, s4.size)
    assert L.index_words == O.index_words(ntr, ntc) and L.bytes_index == 4 * L.index_words


def test_packer_on_tiny_config_and_single_width_bitmaps():
    p = W.make_problem("tiny", 512, 512, 1, 1000)
    L, s2, s3, s4, index = S.sfmp_pack(p.codes, p.bitmap)
    ref = O.pack(p.codes, p.bitmap)
    assert np.array_equal(np.concatenate([s2, s3, s4]), np.concatenate([ref["s2"], ref["s3"], ref["s4"]]))
    for b in (2, 3, 4):
        bitmap = np.full((2, 2), b, dtype=np.int8)
        q = W.make_problem("u", 256, 256, 1, 5 + b, bitmap=bitmap)
        L, s2, s3, s4, index = S.sfmp_pack(q.codes, bitmap)
        ref = O.pack(q.codes, bitmap)
        assert np.array_equal(index, ref["index"])
        for a, name in ((s2, "s2"), (s3, "s3"), (s4, "s4")):
            assert np.array_equal(a, ref[name])
        assert [L.count2, L.count3, L.count4][b - 2] == 4


def test_error_codes():
    lib = S.load_library()
    L = S.SfmpLayout()
    bm = np.full((1, 1), 3, dtype=np.int8)
    ptr = bm.ctypes.data_as(C.c_void_p)
    assert lib.sfmp_pack_query(None, 128, 128, C.byref(L)) == -1  # NULL
    assert lib.sfmp_pack_query(ptr, 100, 128, C.byref(L)) == -2  # SHAPE
    assert lib.sfmp_pack_query(ptr, 128, 0, C.byref(L)) == -2
    bad = np.full((1, 1), 5, dtype=np.int8)
    assert lib.sfmp_pack_query(bad.ctypes.data_as(C.c_void_p), 128, 128, C.byref(L)) == -3  # BITWIDTH
    bad[0, 0] = 1
    assert lib.sfmp_pack_query(bad.ctypes.data_as(C.c_void_p), 128, 128, C.byref(L)) == -3
    # code out of range: nothing written
    codes = np.zeros((128, 128), dtype=np.uint8)
    codes[77, 3] = 8
    with pytest.raises(S.SfmpError) as ei:
        S.sfmp_pack(codes, bm)
    assert ei.value.code == -4
    # workspace query argument checks
    L = S.sfmp_pack_query(bm, 128, 128)
    n = C.c_int64(0)
    assert lib.sfmp_gemm_workspace(C.byref(L), 0, C.byref(n)) == -2
    assert lib.sfmp_gemm_workspace(None, 1, C.byref(n)) == -1
    broken = S.SfmpLayout.from_buffer_copy(L)
    broken.count3 = 7
    assert lib.sfmp_gemm_workspace(C.byref(broken), 1, C.byref(n)) == -8  # LAYOUT
    assert S.sfmp_gemm_workspace(L, 1) >= 256 and S.sfmp_gemm_workspace(L, 1) % 256 == 0
    # gemm refuses NULL buffers before touching any device
    assert lib.sfmp_gemm(None, 1, None, C.byref(L), None, None, None, None, None, None, None, None, None, None, 0,
                         None) == -1
    # alignment is checked before any device work as well (the pointers are never dereferenced on the host)
    ok = [C.c_void_p(0x7f0000001000 + 0x10000 * i) for i in range(8)]

    def gemm_with(X=ok[0], cp=ok[1], scales=ok[2], Y=ok[3], M=1):
        return lib.sfmp_gemm(X, M, cp, C.byref(L), None, ok[4], None, ok[5], scales, ok[6], None, None, Y, ok[7], 1 << 20,
                             None)
    assert gemm_with(X=C.c_void_p(0x7f0000001008)) == -9  # ALIGN: X needs 16 bytes
    assert gemm_with(cp=C.c_void_p(0x7f0000011004)) == -9
    assert gemm_with(scales=C.c_void_p(0x7f0000021002)) == -9
    assert gemm_with(Y=C.c_void_p(0x7f0000031001)) == -9      # Y: 2 bytes at M <= 16 ...
    assert gemm_with(Y=C.c_void_p(0x7f0000031002), M=17) == -9  # ... 16 bytes beyond
    for code in range(-10, 1):
        assert S.sfmp_strerror(code)
    assert "unknown" in S.sfmp_strerror(-99)


def test_check_perm():
    assert S.sfmp_check_perm(np.array([2, 0, 1], dtype=np.int32)) == 0
    assert S.sfmp_check_perm(np.array([2, 0, 2], dtype=np.int32)) == -7
    assert S.sfmp_check_perm(np.array([0, 3, 1], dtype=np.int32)) == -7
    assert S.sfmp_check_perm(np.array([0, -1, 1], dtype=np.int32)) == -7


def test_layout_set_quant_accepts_the_documented_formats_only():
    bitmap = np.full((1, 4), 3, dtype=np.int8)  # N = 128, K = 512
    L = S.sfmp_pack_query(bitmap, 128, 512)
    assert (L.group, L.scale_format) == (128, 0)
    for group in (64, 128, 256, 512):
        for fmt, code in (("fp16", 0), ("bf16", 1)):
            S.sfmp_layout_set_quant(L, group, fmt)
            assert (L.group, L.scale_format) == (group, code)
    S.sfmp_layout_set_quant(L, 128, "fp16")
    lib = S.load_library()
    for group, fmt in ((32, 0), (1024, 0), (384, 0), (128, 2), (256, -1)):
        assert lib.sfmp_layout_set_quant(C.byref(L), group, fmt) == -8
        assert (L.group, L.scale_format) == (128, 0)  # a rejected call leaves the layout alone
    # K must be a multiple of the group
    L3 = S.sfmp_pack_query(np.full((1, 3), 2, dtype=np.int8), 128, 384)
    assert lib.sfmp_layout_set_quant(C.byref(L3), 256, 0) == -8
    assert lib.sfmp_layout_set_quant(None, 128, 0) == -1


def test_fold_perms_matches_oracle_and_its_defining_property():
    # NEXT: permutation folding.  The C ABI result equals the oracle's (written as a search), and both satisfy
    # the property that defines them: gathering from the reordered product with the folded permutation fetches
    # what the plain gather fetches from the un-permuted one.
    import paper_2602_01027_amd as S
    from oracle import sfmp_oracle as O
    rng = np.random.default_rng(5)
    for n in (1, 7, 128, 1000):
        r = rng.permutation(n).astype(np.int32)
        c = rng.permutation(n).astype(np.int32)
        f = S.sfmp_fold_perms(r, c)
        assert np.array_equal(f, O.fold_perms(r, c))
        Y = rng.standard_normal((3, n))
        Yt = Y[:, r]                      # the product left in reordered row order
        assert np.array_equal(Yt[:, f], Y[:, c])
        f_id = S.sfmp_fold_perms(r, None)
        assert np.array_equal(f_id, O.fold_perms(r, None))
        assert np.array_equal(Yt[:, f_id], Y)  # identity next permutation: the fold is the inverse
    assert S.sfmp_check_perm(f) == 0
    with pytest.raises(S.SfmpError):
        S.sfmp_fold_perms(np.array([0, 0, 1], dtype=np.int32), None)
    with pytest.raises(S.SfmpError):
        S.sfmp_fold_perms(np.array([0, 2, 1], dtype=np.int32), np.array([0, 3, 1], dtype=np.int32))


def _plan_mirror(N, K, M):
    """The documented path selection of sfmp_gemm, restated: which kernels a call takes and the workspace it needs."""
    ntr, ntc = N // 128, K // 128
    up256 = lambda v: (v + 255) // 256 * 256
    if M <= 16:
        if M == 1 and K <= 32768 - 1:  # the GEMV kernel holds the activation vector in LDS: no workspace
            return "gemv", None
        mb = 4 if M <= 4 else 8 if M <= 8 else 16
        # a wavefront with at most four tile columns keeps the activations in registers (staged as 16 rows), unless
        # the kernel stages M <= 4 rows into LDS by itself (at most 32 KiB of them)
        grid = min(8 * ntr, 256)
        for rounds in (2, 3, 4):  # up to four workgroups per CU in turn, to get down to 8 slabs per workgroup
            if -(-8 * ntr // grid) > 8 and -(-8 * ntr // (256 * rounds)) <= 8:
                grid = 256 * rounds
        if -(-8 * ntr // grid) > 16:
            grid = (-(-8 * ntr // 16) + 7) // 8 * 8
        max_slabs = -(-8 * ntr // grid)
        nw = 16 if max_slabs <= 8 else 8
        resident = mb == 4 and M * K * 2 <= 32 * 1024 and K // 8 <= 4 * nw * 64
        # (that form keeps each wavefront's finished sums in LDS, 1 KiB per slab, beside two ring slots of 1280 bytes)
        if not resident and ntc <= 4 * nw and nw * (max_slabs * 1024 + 2 * 1280) <= 160 * 1024:
            mb = 16
        return "ring", up256(ntc * mb * 256)
    chunks = (M + 15) // 16
    if ntr <= 8:
        chunked = chunks <= 8
    elif ntc <= 64:  # K <= 8192: the chunks keep their activations in registers
        tiles = ntr * ntc
        chunked = chunks <= 2 or (chunks <= 4 and tiles <= 1536) or (chunks <= 6 and tiles <= 1024)
    else:
        chunked = chunks <= 2 and ntr <= 32
    if M <= 128 and ntc >= 32 and chunked:
        return "chunked", chunks * up256(ntc * 16 * 256)
    bm = 64 if ((M + 127) // 128) * ntr <= 128 else 128
    blocks = ((M + bm - 1) // bm) * ntr
    ks = 1
    if blocks <= 256:
        ks = max(1, min(512 // blocks, ntc // 8, 8))
        if ks < 3 and ntc < 64:
            ks = 1
    xperm = up256(((M + 127) // 128) * 128 * K * 2)
    ytmp = up256(ks * M * N * 4 if ks > 1 else M * N * 2)
    return f"mfma bm={bm} ksplit={ks}", xperm + ytmp


@pytest.mark.parametrize("N,K,M", [(4096, 4096, 4), (4096, 4096, 3), (14336, 4096, 5), (32768, 4096, 2), (57344, 4096, 8), (57344, 8192, 8), (4096, 8192, 3), (4096, 14336, 16), (1024, 4096, 128), (1152, 4096, 128),
                                    (4096, 4096, 32), (4096, 4096, 33), (4096, 4096, 96), (4096, 4096, 97), (6144, 4096, 64), (14336, 4096, 32),
                                    (14336, 4096, 33), (8192, 8192, 32), (8192, 8192, 48), (28672, 8192, 32), (4096, 14336, 32), (4096, 14336, 256), (14336, 4096, 48),
                                    (14336, 4096, 256), (4096, 4096, 2048), (28672, 8192, 2048), (4096, 2048, 100),
                                    (8192, 28672, 512)])
def test_workspace_query_follows_the_documented_path_selection(N, K, M):
    bitmap = np.full((N // 128, K // 128), 3, dtype=np.int8)
    L = S.sfmp_pack_query(bitmap, N, K)
    name, expected = _plan_mirror(N, K, M)
    got = S.sfmp_gemm_workspace(L, M)
    if expected is not None:
        assert got == max(256, expected), (name, got, expected)
    else:
        assert got == 256, (name, got)


# ---- bit-plane format of the lookup-table GEMV: the library's packer against the oracle's, byte for byte ----------
@pytest.mark.parametrize("seed,N,K,fractions", [(21, 128, 128, {4: 1.0}), (22, 256, 384, None), (23, 384, 256, {2: 0.6, 3: 0.4})])
def test_lut_pack_bytes_match_oracle(seed, N, K, fractions):
    from oracle import sfmp_lut_oracle as LO
    p = W.make_problem("lutpack", K, N, 1, seed, fractions=fractions)
    planes, tile_off = S.sfmp_lut_pack(p.codes, p.bitmap)
    ref_planes, ref_off = LO.lut_pack(p.codes, p.bitmap)
    assert np.array_equal(tile_off, ref_off)
    assert np.array_equal(planes, ref_planes)
    assert np.array_equal(LO.lut_unpack(N, K, planes, tile_off), p.codes)


def test_lut_pack_errors():
    codes = np.zeros((128, 128), dtype=np.uint8)
    with pytest.raises(S.SfmpError) as e:
        S.sfmp_lut_pack(codes, np.array([[5]], dtype=np.int8))
    assert e.value.code == -3
    codes[3, 7] = 4
    with pytest.raises(S.SfmpError) as e:
        S.sfmp_lut_pack(codes, np.array([[2]], dtype=np.int8))
    assert e.value.code == -4
    with pytest.raises(S.SfmpError) as e:
        S.sfmp_lut_pack(np.zeros((100, 128), dtype=np.uint8), np.array([[2]], dtype=np.int8))
    assert e.value.code == -2
    assert S.sfmp_lut_gemv_workspace(4096, 4096) % 256 == 0


def test_float_reciprocal_item_index_is_exact():
    """The decode kernels find the slab index of an item as floor((e + 0.5) * rcp(c)) in fp32 instead of an integer
    division (e < 1024 items, c <= 64 tile columns per wavefront).  Exact even if the hardware reciprocal is off by
    two units in the last place in either direction."""
    e = np.arange(1024)
    g = e.astype(np.float32) + np.float32(0.5)
    for c in range(1, 65):
        r = np.float32(1) / np.float32(c)
        lo = np.nextafter(np.nextafter(r, np.float32(0)), np.float32(0))
        hi = np.nextafter(np.nextafter(r, np.float32(2)), np.float32(2))
        for rr in (lo, r, hi):
            j = (g * np.float32(rr)).astype(np.uint32)
            assert np.array_equal(j, e // c), c


@pytest.mark.parametrize("odd", ["host tensor", "no tensor", "layout", "short tuple", "nine"])
def test_launcher_leaves_calls_that_are_not_plain_to_the_general_path(odd):
    # the extension answers None (nothing launched) for what is no plain call; the ctypes path then raises what it always
    # raised.  (Each reason alone, with everything else valid, takes device tensors: tests/test_gpu_parity.py.)
    import types
    import torch
    module = S.binding._launcher()
    L = S.sfmp_pack_query(np.full((1, 1), 3, dtype=np.int8), 128, 128)
    t, stream = torch.zeros((1, 128), dtype=torch.float16), types.SimpleNamespace(cuda_stream=0)
    gemm_args = [t, None, L, t, t, t, t, t, t, t, None, t, t, stream]
    dp = S.DevicePacked(L, t, t, t, t, t, t, t)
    if odd in ("host tensor", "layout", "no tensor"):
        gemm_args[0] = 3 if odd == "no tensor" else t
        gemm_args[2] = 7 if odd == "layout" else L
        assert module.gemm(*gemm_args) is None
        assert module.gemm_static(*gemm_args[:12], stream) is None
    else:
        q = {"short tuple": [(t, None, dp, None)], "nine": [(t, None, dp, None, t)] * 9}[odd]
        assert module.gemv_batched(q, stream) is None
        assert module.gemm_batched(q, 2, t, stream) is None


@pytest.mark.parametrize("entry", ["gemv_batched", "gemm_batched"])
@pytest.mark.parametrize("when", ["attribute", "stream", "library", "made by the access"])
def test_launcher_keeps_the_arguments_of_a_batch_alive(entry, when):
    # The list of problems is emptied during the call: by an attribute lookup of the call itself, by the stream object's
    # property, or while the library runs (without the GIL, where any other thread may do it).  What the library was given
    # has to stay alive and unchanged until it returns; so has an attribute that its access makes and nobody else keeps.
    import gc
    import weakref
    import torch
    module = S.binding._launcher()
    lib = S.load_library()
    expected = bytes(S.sfmp_pack_query(np.full((2, 1), 3, dtype=np.int8), 256, 128))
    seen, problems, refs = [], [], []

    def drop(at):
        if at == when:
            problems.clear()
            gc.collect()

    class Packed(S.DevicePacked):
        def __getattribute__(self, name):
            if name == "s3":
                drop("attribute")
            if name == "bitmap" and when == "made by the access":
                made = torch.zeros(128)
                refs.append(weakref.ref(made))
                return made
            return super().__getattribute__(name)

    class Stream:
        @property
        def cuda_stream(self):
            drop("stream")
            return 0

    def fill():
        t = lambda: torch.zeros((1, 128), dtype=torch.float16)
        for _ in range(2):
            layout = S.sfmp_pack_query(np.full((2, 1), 3, dtype=np.int8), 256, 128)
            x, packed, y = t(), Packed(layout, *(t() for _ in range(7))), t()
            refs.extend(weakref.ref(o) for o in (layout, packed, x, y))
            problems.append((x, None, packed, None, y))

    def library(array, count, *_rest):
        drop("library")
        seen.append(([r() is not None for r in refs], count,
                     [C.string_at(S.binding.SfmpGemvProblem.from_address(array + i * C.sizeof(S.binding.SfmpGemvProblem)).layout, 72)
                      for i in range(count)]))
        return 0

    fill()
    int32, vp = C.c_int32, C.c_void_p
    ours = (C.CFUNCTYPE(int32, vp, int32, vp)(library) if entry == "gemv_batched" else
            C.CFUNCTYPE(int32, vp, int32, int32, vp, C.c_int64, vp)(library))
    addresses = [C.cast(f, vp).value for f in (lib.sfmp_gemm, lib.sfmp_gemm_static, lib.sfmp_gemv_batched, lib.sfmp_gemm_batched)]
    replaced = list(addresses)
    replaced[2 if entry == "gemv_batched" else 3] = C.cast(ours, vp).value
    bind = lambda a: module.bind(S.SfmpLayout, torch._C._cuda_getDevice, torch._C._cuda_getCurrentRawStream, *a)
    bind(replaced)
    try:
        if entry == "gemv_batched":
            rc = module.gemv_batched(problems, Stream())
        else:
            rc = module.gemm_batched(problems, 2, torch.zeros(256, dtype=torch.uint8), Stream())
    finally:
        bind(addresses)
    assert rc == 0 and (problems == [] or when == "made by the access")
    assert seen == [([True] * len(refs), 2, [expected] * 2)] and len(refs) == (10 if when == "made by the access" else 8)
    problems.clear()
    assert not any(r() is not None for r in refs)  # and no longer than that


@pytest.mark.parametrize("extension", ["built", "missing", "not loadable", "built for another torch"])
def test_launches_without_a_usable_extension_take_the_ctypes_path(extension, tmp_path, monkeypatch):
    # the extension reads torch's objects by the layout of the headers it was built with: where it cannot be loaded or was
    # built for another torch, the entry points say so and reach the library through ctypes
    import types
    import warnings
    import torch
    B = S.binding
    monkeypatch.setattr(B, "_LAUNCHER", None)
    path = tmp_path / "_sfmp_torch.so"
    if extension == "not loadable":
        path.write_bytes(b"not a shared object")
    if extension in ("missing", "not loadable"):
        monkeypatch.setattr(B, "launcher_path", lambda: str(path))
    if extension == "built for another torch":
        monkeypatch.setattr(torch, "__version__", "1.0")
    L = S.sfmp_pack_query(np.full((1, 1), 3, dtype=np.int8), 128, 128)
    empty, stream = torch.empty((1, 0), dtype=torch.float16), types.SimpleNamespace(cuda_stream=0)
    with warnings.catch_warnings(record=True) as caught:
        warnings.simplefilter("always")
        # (null buffers: refused by the library before it touches a device)
        for call in (lambda: S.sfmp_gemm(empty, None, L, *[empty] * 7, None, empty, empty, stream=stream),
                     lambda: S.sfmp_gemm_static(empty, None, L, *[empty] * 7, None, empty, stream=stream),
                     lambda: S.sfmp_gemv_batched([(empty, None, S.DevicePacked(L, *[empty] * 7), None, empty)], stream=stream),
                     lambda: S.sfmp_gemm_batched([(empty, None, S.DevicePacked(L, *[empty] * 7), None, empty)], 2, empty,
                                                 stream=stream)):
            with pytest.raises(S.SfmpError) as e:
                call()
            assert e.value.code == -1
    assert len([w for w in caught if "marshalled by ctypes" in str(w.message)]) == (0 if extension == "built" else 1)
    assert (B._LAUNCHER[1] is B._NoExtension) == (extension != "built")


def test_workspace_of_a_matrix_core_call_is_the_documented_one():
    import plan_util
    rng = np.random.default_rng(11)
    for _ in range(4000):
        K, N = (int(128 * np.ceil(2 ** rng.uniform(0, 7.8))) for _ in range(2))
        M = int(2 ** rng.uniform(4.1, 11))
        if not plan_util.chunked(N, K, M):
            assert sum(plan_util.prefill_bytes(N, K, M)) == _plan_mirror(N, K, M)[1], (N, K, M)


def test_launched_form_of_a_matrix_core_call():
    # at least one tile per K group, at most the documented ranges, the plain kernel only with more than 256 blocks of 128 rows
    import plan_util
    rng = np.random.default_rng(12)
    for _ in range(4000):
        K, N = (int(128 * np.ceil(2 ** rng.uniform(0, 7.8))) for _ in range(2))
        M = int(2 ** rng.uniform(4.1, 11))
        if plan_util.chunked(N, K, M):
            continue
        mi, kg, ksplit = plan_util.launched_form(N, K, M)
        documented = int(_plan_mirror(N, K, M)[0].split("ksplit=")[1])
        assert (mi == 0 and (kg, ksplit) == (1, 1) and -(-M // 128) * (N // 128) > 256) or 4 <= mi <= 8, (N, K, M)
        assert 1 <= ksplit <= documented and kg * ksplit <= K // 128, (N, K, M)
        assert ksplit == 1 or (kg == 2 and ksplit * M * N * 4 <= plan_util.prefill_bytes(N, K, M)[1]), (N, K, M)
    for shape, form in (((4096, 4096, 777), (7, 2, 1)), ((14336, 4096, 64), (4, 2, 2)), ((4096, 14336, 200), (7, 2, 4)),
                        ((14336, 4096, 2048), (8, 1, 1)), ((8192, 28672, 2048), (8, 1, 1)), ((128, 128, 17), (4, 1, 1)),
                        ((4480, 19968, 295), (7, 2, 2)), ((512, 8832, 152), (4, 2, 7)), ((1152, 14336, 214), (4, 2, 7)), ((1152, 13824, 391), (5, 2, 5)),
                        ((1024, 13824, 384), (4, 2, 5))):
        assert plan_util.launched_form(*shape) == form, shape


def test_chunks_without_staging_touch_no_workspace():
    # whatever the mix of widths and the group length: the whole launch takes the form whose operands the kernel gathers itself
    import plan_util
    rng = np.random.default_rng(13)
    taken = 0
    for _ in range(300):
        K, N = (int(128 * np.ceil(2 ** rng.uniform(0, hi))) for hi in (5.2, 7.5))
        M, group = int(rng.integers(15, 132)), int(rng.choice((64, 128)))
        if not plan_util.chunks_without_staging(N, K, M, group):
            continue
        taken += 1
        layout = S.sfmp_layout_set_quant(S.sfmp_pack_query(rng.integers(2, 5, (N // 128, K // 128)).astype(np.int8), N, K), group, "fp16")
        config, grids = plan_util.batched_config([layout] * -(-M // 16), 16)
        assert 17 <= M <= 128 and K <= 4096 and config.ra == 2 and config.resident, (N, K, M)
        assert max(-(-N // 16 // g) for g in grids) <= 7, (N, K, M)
    assert taken > 60


def test_outputs_over_activations_are_staged_first():
    # a launch whose workgroups gather their own activations may not store a row that another one has yet to read: where an
    # output overlaps activations (its own problem's or another's) they are staged in a launch of their own, as for M >= 5 on any
    # other matrix
    import plan_util
    at = 0x7f0000000000
    for M, group, n in ((5, 128, 1), (16, 128, 3), (3, 64, 2)):
        layouts = [S.sfmp_layout_set_quant(S.sfmp_pack_query(np.full((N // 128, 16), 3, dtype=np.int8), N, 2048), group, "fp16")
                   for N in (2048, 1024, 4096)[:n]]
        nx, ny = M * 2048 * 2, [M * layout.N * 2 for layout in layouts]
        apart_x, apart_y = [at + i * 2 ** 20 for i in range(n)], [at + (8 + i) * 2 ** 20 for i in range(n)]
        last = n - 1
        for x0, y, gathered in ((at, apart_y, True), (at, [*apart_y[:last], at + nx], True), (at, [*apart_y[:last], at - ny[last]], True),
                                (at, [*apart_y[:last], at], False), (at, [*apart_y[:last], at + nx - 2], False),
                                (at, [*apart_y[:last], at - ny[last] + 2], False)):
            c = plan_util.batched_config(layouts, M, [x0, *apart_x[1:]], y)[0]
            assert (c.ra, c.resident) == (2, gathered), (M, group, [hex(v) for v in y])
            if n == 1:
                d = plan_util.launched_decode_plan(layouts[0], M, x0, y[0])
                assert (d.ra, d.resident) == (2, gathered) and d.lds_bytes <= 160 * 1024
                assert d.workspace_bytes == plan_util.decode_plan(layouts[0].N, 2048, M, group).workspace_bytes
    # 17 to 128 rows beyond the documented chunked shapes: the matrix-core path, which stages them
    layout = S.sfmp_pack_query(np.full((4, 4), 3, dtype=np.int8), 512, 512)
    assert plan_util.chunks_without_staging(512, 512, 64)
    assert plan_util.runs_in_chunks(layout, 64, at, at + 2 ** 20) and not plan_util.runs_in_chunks(layout, 64, at, at + 16)


@pytest.mark.parametrize("N,K,M,both", [
    (6272, 4096, 53, False), (3328, 4096, 97, False), (7168, 4096, 49, False), (6528, 4096, 55, False),  # 5 to 11 % slower in chunks
    (7168, 2048, 49, True), (4096, 2048, 32, True), (512, 512, 64, True), (14208, 1024, 20, True)])
def test_chunks_without_staging_by_group_length(N, K, M, both):
    # two parameter pairs per tile column make chunks slower: with many slabs and a long K the matrix-core path is the faster one
    import plan_util
    assert plan_util.chunks_without_staging(N, K, M, 128) and plan_util.chunks_without_staging(N, K, M, 64) == both


@pytest.mark.parametrize("N,K,M,gathered", [
    (32768, 4096, 16, None), (28672, 4096, 16, True), (32896, 4096, 16, False), (32896, 3072, 16, True), (32896, 4096, 8, True),
    (57344, 3200, 9, False), (65664, 2176, 9, False), (65664, 2048, 16, True), (65664, 4096, 8, True)])
def test_activations_are_gathered_where_the_start_is_paid_for_seldom(N, K, M, gathered):
    # more than 8 rows: one round of workgroups (up to 7 slabs each), two with K <= 3072, more with K <= 2048; staged beyond
    import plan_util
    d = plan_util.decode_plan(N, K, M)
    assert (d.ra, d.resident) == ((0, False) if gathered is None else (2, gathered))
    assert d.workspace_bytes == K // 128 * 16 * 256


@pytest.mark.parametrize("N,K,M,group,streamed", [
    (8192, 28672, 8, 128, True), (8192, 28672, 16, 64, True), (4224, 8320, 5, 128, True), (8192, 8320, 16, 64, True),
    (8192, 12288, 8, 64, True), (8192, 12160, 8, 64, False),  # up to 8 rows, group length 64: from K = 12288 on
    (4096, 14336, 16, 128, False), (8192, 28672, 4, 128, False), (8192, 8192, 16, 128, False), (8320, 14336, 16, 128, False)])
def test_small_batches_that_stream_their_activations(N, K, M, group, streamed):
    import plan_util
    assert plan_util.decode_plan(N, K, M, group).rs == (2 if streamed else 0)


@pytest.mark.parametrize("N,M,past", [
    (14336, 2048, False), (4096, 777, False), (8192, 150, False), (28672, 2048, False),  # shorter alone, longer with the reader of the result
    (4096, 16383, False), (4096, 16384, True), (28672, 4096, True)])
def test_result_of_a_prompt_goes_past_the_caches_only_where_they_could_not_hold_it(N, M, past):
    import plan_util
    assert plan_util.stores_past_caches(N, M) == past


@pytest.mark.parametrize("N,M,threads", [
    (10240, 777, 256), (10240, 512, 256), (6144, 520, 256), (128, 2048, 256),  # longer with more threads
    (10368, 512, 704), (10240, 511, 1024), (8192, 150, 1024), (4096, 300, 512), (128, 130, 64), (28672, 2048, 896), (81920, 130, 1024)])
def test_threads_of_the_un_permute_pass(N, M, threads):
    import plan_util
    assert plan_util.scatter_threads(N, M) == threads


@pytest.mark.parametrize("N,K,M,tail", [
    (6784, 1792, 1524, (0, 0)), (6912, 6016, 1354, (0, 0)),  # 33 pieces for an XCD whose 32 CUs all have a large workgroup: two rounds
    (14336, 4096, 2048, (8, 16)), (13184, 640, 2047, (4, 7)), (5632, 9088, 1681, (4, 8))])
def test_tail_of_a_prompt_counts_its_rounds_per_xcd(N, K, M, tail):
    import plan_util
    assert plan_util.launched_tail(N, K, M) == tail


def test_prompts_with_a_tail_have_no_k_ranges():
    # the workgroups of both sizes go over the whole K: partial products of the form in one size would never be summed
    import plan_util
    rng = np.random.default_rng(14)
    tails = 0
    for _ in range(6000):
        K, N = (int(128 * np.ceil(2 ** rng.uniform(2, 7.8))) for _ in range(2))
        M = int(rng.integers(257, 2049))
        mi, tile_rows = plan_util.launched_tail(N, K, M)
        if mi:
            tails += 1
            assert 0 < tile_rows < N // 128 and plan_util.launched_form(N, K, M)[2] == 1, (N, K, M)
    assert tails > 100
