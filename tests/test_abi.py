"""CPU-side checks of the boundary: the library builds, loads and exports every
symbol that include/heart.h and include/heart_diag.h declare, and host-side validation
rejects bad calls before anything touches a GPU."""
import ctypes
import os
import re

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def lib():
    from paper_2605_14513_amd import build as hb
    from paper_2605_14513_amd import binding

    if hb.is_stale():
        hb.build(force=True)
    return binding.load_library()


def declared_symbols(headers=("heart.h", "heart_diag.h")):
    syms = set()
    for h in headers:
        text = open(os.path.join(ROOT, "include", h)).read()
        text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
        syms |= set(re.findall(r"\b(heart_[a-z_0-9]+)\s*\(", text))
    return sorted(syms)


def test_header_declares_the_four_hot_path_calls():
    syms = declared_symbols(("heart.h",))
    for s in ("heart_pool_qk", "heart_drift", "heart_mask_topp", "heart_block_sparse_attn",
              "heart_workspace_bytes", "heart_last_error", "heart_version"):
        assert s in syms
    # diagnostics live in their own header
    assert not [s for s in syms if "ubench" in s]
    assert "heart_ubench_read" in declared_symbols(("heart_diag.h",))


def test_library_exports_every_declared_symbol(lib):
    for s in declared_symbols():
        assert hasattr(lib, s), f"libheart.so does not export {s}"
    assert lib.heart_version() >= 100


def test_binding_names_match_header():
    import paper_2605_14513_amd as pkg

    for s in declared_symbols():
        assert hasattr(pkg, s), f"python binding lacks {s}"


def test_shape_struct_layout_matches_header():
    from paper_2605_14513_amd.binding import HeartShape

    # 5 ints (20 bytes, padded to 24) + 4 * 3 long long
    assert ctypes.sizeof(HeartShape) == 24 + 4 * 3 * 8
    assert HeartShape.q_stride.offset == 24 and HeartShape.o_stride.offset == 24 + 72


def test_host_validation_rejects_bad_calls_without_a_gpu(lib):
    from paper_2605_14513_amd.binding import HeartShape

    assert lib.heart_pool_qk(None, None, None, None, None, None, None, None) == -1
    assert b"shape is NULL" in lib.heart_last_error()
    s = HeartShape()
    s.B, s.H, s.N, s.D, s.block = 1, 2, 100, 96, 128
    assert lib.heart_pool_qk(ctypes.byref(s), None, None, None, None, None, None, None) == -2
    assert b"D must be 64 or 128" in lib.heart_last_error()
    s.D = 128
    assert lib.heart_pool_qk(ctypes.byref(s), None, None, None, None, None, None, None) == -1
    s.block = 100
    assert lib.heart_block_sparse_attn(ctypes.byref(s), None, None, None, None, None, 0.0, None,
                                       None, None, 0, None) == -2
    s.block = 128
    assert lib.heart_attn_workspace_bytes(ctypes.byref(s)) == (1 * 2 * (1 + 2) + 24) * 4
    assert lib.heart_attn_workspace_bytes(None) == 0
    assert lib.heart_workspace_bytes(1, 2, 1, 128) == (1 * 2 * (1 + 2) + 24) * 4
    assert lib.heart_workspace_bytes(1, 40, 256, 128) == (40 * 258 + 24) * 4
    assert lib.heart_workspace_bytes(0, 2, 1, 128) == 0
    fake = ctypes.c_void_p(0x10000)
    for arr in (s.q_stride, s.k_stride, s.v_stride, s.o_stride):
        arr[0], arr[1], arr[2] = 2 * 100 * 128, 100 * 128, 128
    # unknown option bits are refused before anything is launched
    assert lib.heart_block_sparse_attn_flags(ctypes.byref(s), fake, fake, fake, fake, fake, 0.0, 2,
                                             fake, None, None, 0, None) == -1
    assert b"flag" in lib.heart_last_error()
    assert lib.heart_drift(1, 2, 96, None, None, None, None, None, None, 0.4, 0.8, 1, None, None,
                           None) == -2
    assert lib.heart_drift(1, 2, 64, None, None, None, None, None, None, 0.4, 0.8, 1, None, None,
                           None) == -1
    assert lib.heart_mask_topp(1, 1, 2000, 128, None, None, None, None, None, 0, 0, 1, None, None,
                               None, None, None) == -2
    assert b"HEART_MAX_NB" in lib.heart_last_error()
    assert lib.heart_mask_topp(1, 1, 8, 128, None, None, None, None, None, 0, 0, 1, None, None,
                               None, None, None) == -1


def test_sizes_at_the_ends_of_their_types_without_a_gpu(lib):
    """B*H*Nb that leaves 64 bits is refused, and the workspace sizes of such shapes (and of the largest
    N) can be asked for; none of these calls reaches a GPU."""
    from paper_2605_14513_amd.binding import HeartShape

    s = HeartShape()
    f = ctypes.c_void_p(0x10000)
    for arr in (s.q_stride, s.k_stride, s.v_stride, s.o_stride):
        arr[0], arr[1], arr[2] = 0, 64, 64
    s.D = s.block = 64
    attn = lambda n_bytes: lib.heart_block_sparse_attn(ctypes.byref(s), f, f, f, f, f, 0.0, f, None, f, n_bytes, None)
    # 2^30 * 2^30 heads of 16 or 15 blocks: the number of rows is 2^64 (0 in 64 bits) or 15 * 2^60 (negative)
    for s.N in (1024, 960):
        s.B = s.H = 1 << 30
        assert lib.heart_attn_workspace_bytes(ctypes.byref(s)) > 0
        assert attn((1 << 64) - 1) == -2 and b"grid limit" in lib.heart_last_error()
        assert lib.heart_pool_qk(ctypes.byref(s), f, f, f, f, f, f, None) == -2
        assert lib.heart_mask_topp(s.B, s.H, s.N // 64, 64, f, f, None, f, None, 0, 0, 1, f, f, f, None, None) == -2
    s.B, s.H, s.N = 1, 1, 2 ** 31 - 1
    nb = 2 ** 25  # (N + block - 1 is past 32 bits)
    need = lib.heart_workspace_bytes(1, 1, nb, 64)
    assert need == (nb + 2 + 24) * 4 and lib.heart_attn_workspace_bytes(ctypes.byref(s)) == need + 2304
    assert attn(need - 1) == -1 and str(need).encode() in lib.heart_last_error()
    assert attn(need) == -2 and b"4 GiB" in lib.heart_last_error()
    assert lib.heart_block_sparse_attn_static(ctypes.byref(s), f, f, f, f, f, 0.0, 0, f, None, None) == -2
    assert b"static array" in lib.heart_last_error()


def test_mask_topp_workspace_validation_without_a_gpu(lib):
    f = ctypes.c_void_p(0x10000)
    need = 1 * 40 * 256 * (2 * 4 * 128 + 2 * 4)  # slices of Q and K blocks and their exponents
    assert lib.heart_mask_topp_workspace_bytes(1, 40, 256, 128) == need
    assert lib.heart_mask_topp_workspace_bytes(1, 0, 256, 128) == 0
    args = lambda ws, nbytes: (1, 40, 256, 128, f, f, None, f, None, 0, 0, 1, f, f, f, None, ws, nbytes, None)
    assert lib.heart_mask_topp_ws(*args(f, need - 1)) == -1                     # too small
    assert b"workspace" in lib.heart_last_error()
    assert lib.heart_mask_topp_ws(*args(ctypes.c_void_p(0x10008), need)) == -2  # misaligned
    assert lib.heart_mask_topp_ws(1, 1, 2000, 128, f, f, None, f, None, 0, 0, 1, f, f, f, None, f,
                                  1 << 30, None) == -2                           # the checks of heart_mask_topp
    assert b"HEART_MAX_NB" in lib.heart_last_error()


def test_pool_drift_validation_without_a_gpu(lib):
    from paper_2605_14513_amd.binding import HeartShape

    s = HeartShape()
    s.B, s.H, s.N, s.D, s.block = 2, 40, 1000, 128, 128
    for arr in (s.q_stride, s.k_stride, s.v_stride, s.o_stride):
        arr[0], arr[1], arr[2] = 40 * 1000 * 128, 1000 * 128, 128
    f = ctypes.c_void_p(0x10000)
    args = lambda ws, nbytes, hi=0.8: (ctypes.byref(s), f, f, f, f, f, f, f, f, f, f, 0.4, hi, 1, f, f, ws, nbytes, None)
    assert lib.heart_pool_drift_workspace_bytes(2, 40) == 2 * 4  # one ticket per batch item
    assert lib.heart_pool_drift_workspace_bytes(0, 40) == 0
    assert lib.heart_pool_drift(*args(None, 8)) == -1                     # no workspace
    assert lib.heart_pool_drift(*args(f, 4)) == -1                        # too small
    assert b"workspace" in lib.heart_last_error()
    assert lib.heart_pool_drift(*args(ctypes.c_void_p(0x10002), 8)) == -2  # misaligned
    assert lib.heart_pool_drift(*args(f, 8, hi=0.1)) == -1                # gate_lo > gate_hi
    s.H = 5000
    assert lib.heart_pool_drift(*args(f, 1 << 20)) == -2                  # more heads than the drift stage holds


def test_estimator_validation_without_a_gpu(lib):
    """heart_scores_antidiag checks shape, stride relation, pointers, alignment and workspace
    size on the host; the pointers below are never dereferenced."""
    from paper_2605_14513_amd.binding import HeartShape

    s = HeartShape()
    s.B, s.H, s.N, s.D, s.block = 1, 2, 1000, 128, 128
    for arr in (s.q_stride, s.k_stride, s.v_stride, s.o_stride):
        arr[0], arr[1], arr[2] = 2 * 1000 * 128, 1000 * 128, 128
    fake = ctypes.c_void_p(0x10000)
    call = lib.heart_scores_antidiag
    assert call(None, fake, fake, 16, None, fake, fake, 1 << 30, None) == -1
    assert call(ctypes.byref(s), fake, fake, 8, None, fake, fake, 1 << 30, None) == -2
    assert b"8 * stride" in lib.heart_last_error()
    assert call(ctypes.byref(s), None, fake, 16, None, fake, fake, 1 << 30, None) == -1
    assert call(ctypes.byref(s), ctypes.c_void_p(0x10008), fake, 16, None, fake, fake, 1 << 30, None) == -2
    need = lib.heart_scores_antidiag_workspace_bytes(ctypes.byref(s), 16)
    # 63 reduced rows -> one 256-row tile -> 2 records of 128 keys: 16 * 2 sums + 2 maxima per row
    assert need == 1 * 2 * 63 * (32 + 2) * 4
    assert call(ctypes.byref(s), fake, fake, 16, None, fake, fake, need - 1, None) == -1
    assert b"workspace" in lib.heart_last_error()
    s.k_stride[2] = 132   # not a multiple of 8 elements
    assert call(ctypes.byref(s), fake, fake, 16, None, fake, fake, need, None) == -2
    s.k_stride[2] = 128
    s.N = 128 * 1025      # more key blocks than the mask kernel ranks
    assert call(ctypes.byref(s), fake, fake, 16, None, fake, fake, 1 << 40, None) == -2
    assert b"HEART_MAX_NB" in lib.heart_last_error()
    assert lib.heart_scores_antidiag_workspace_bytes(None, 16) == 0


def test_binding_refuses_cpu_tensors(lib):
    import torch

    import paper_2605_14513_amd as pkg

    q = torch.zeros((1, 1, 128, 128), dtype=torch.bfloat16)
    with pytest.raises(TypeError):
        pkg.heart_pool_qk(q, q, 128, qblk=torch.zeros(1, 1, 1, 128), kblk=torch.zeros(1, 1, 1, 128),
                          qmean=torch.zeros(1, 1, 128), kmean=torch.zeros(1, 1, 128))


def test_binding_refuses_fractional_blocks(lib):
    import torch

    from paper_2605_14513_amd import binding

    q, x, native = torch.zeros((1, 1, 128, 128), dtype=torch.bfloat16), torch.zeros(1), binding._native()
    for block in (128.0, 128.5):
        with pytest.raises(TypeError, match="block"):
            native.block_sparse_attn(q, q, q, block, x, x, 0.0, 0, q, None, None, 0)
        with pytest.raises(TypeError, match="block"):
            native.pool_drift(q, q, block, x, x, x, x, x, 0.4, 0.8, True, x, x, x, x, x, x, 0)
        with pytest.raises(TypeError, match="block"):
            native.scores_antidiag(q, q, block, 16, x, x, None, 0)


def test_binding_errors_of_empty_divisors(lib):
    """No blocks of no tokens and no empty axes: the division that counts them raises, as it does in Python."""
    import torch

    from paper_2605_14513_amd import binding

    q, x, native = torch.zeros((1, 1, 128, 128), dtype=torch.bfloat16), torch.zeros(1), binding._native()
    with pytest.raises(ZeroDivisionError):
        native.block_sparse_attn(q, q, q, 0, x, x, 0.0, 0, q, None, None, 0)
    with pytest.raises(ZeroDivisionError):
        native.pool_drift(q, q, 0, x, x, x, x, x, 0.4, 0.8, True, x, x, x, x, x, x, 0)
    with pytest.raises(ZeroDivisionError):
        native.scores_antidiag(q, q, 0, 16, x, x, None, 0)
    with pytest.raises(ValueError, match="kept_idx"):  # (no list has a negative number of blocks)
        native.block_sparse_attn(q, q, q, -128, torch.zeros((1, 1, 1, 1)), torch.zeros((1, 1, 1)), 0.0, 0, q, None, None, 0)
    e = torch.zeros((2, 0, 4, 5))
    with pytest.raises(ZeroDivisionError):
        native.ebc_band_error(e, e, 1.0, 1.0, 1.0, 1.0, 1e-8, x, torch.zeros(6, dtype=torch.float64), 0)


def test_binding_refuses_tensors_that_are_too_small(lib):
    """What a kernel writes or reads has to be there (sizes are checked before devices are)."""
    import torch

    from paper_2605_14513_amd import binding

    native = binding._native()
    B, H, N, D, Nb = 2, 3, 300, 64, 3
    bf = dict(dtype=torch.bfloat16)
    q = torch.zeros((B, H, N, D), **bf)
    idx, cnt = torch.zeros((B, H, Nb, Nb), dtype=torch.int32), torch.zeros((B, H, Nb), dtype=torch.int32)

    def attn(out):
        native.block_sparse_attn(q, q, q, 128, idx, cnt, 0.0, 0, out, None, None, 0)

    for shape in ((B, H, N - 1, D), (B, H - 1, N, D), (1, H, N, D), (B, H, N, D // 2)):
        with pytest.raises(ValueError, match="out"):
            attn(torch.zeros(shape, **bf))
    with pytest.raises(TypeError, match="GPU"):  # (room for more is no fault: the device is the next one)
        attn(torch.zeros((B, H, N + 5, D), **bf))

    blk, mean, bh = torch.zeros((B, H, Nb, D)), torch.zeros((B, H, D)), torch.zeros((B, H), dtype=torch.uint8)
    drift, delta, few = torch.zeros((B, H)), torch.zeros(H), torch.zeros((B, H, Nb - 1, D))
    for qblk, kblk in ((few, blk), (blk, few)):
        with pytest.raises(ValueError, match="blk must hold"):
            native.pool_drift(q, q, 128, mean, mean, bh, delta, bh, 0.4, 0.8, True, qblk, kblk, mean, mean, drift, bh, 0)
        with pytest.raises(ValueError, match="blk must hold"):
            binding.heart_pool_qk(q, q, 128, qblk, kblk, mean, mean)
    for qmean, kmean in ((mean[:1], mean), (mean, mean[:1])):
        with pytest.raises(ValueError, match="mean must hold"):
            binding.heart_pool_qk(q, q, 128, blk, blk, qmean, kmean)

    with pytest.raises(ValueError, match="scores_in"):
        native.mask_topp(None, None, delta, None, torch.zeros((B, H, Nb, Nb - 1)), 0, 0, 1, idx, idx, cnt, None, None, 0)

    x = torch.zeros((2, 3, 4, 5))
    with pytest.raises(ValueError, match="out"):
        native.ebc_band_error(x, x, 1.0, 1.0, 1.0, 1.0, 1e-8, x, torch.zeros(5, dtype=torch.float64), 0)


# (B, H, Nb, D, block): a size of its own asks for divided rows, or there is none.  Parts of split rows with few blocks are left as
# they are: 15 a part in two parts or at blocks of 128, 30 at D = 64 and 24 at D = 128 in more parts
@pytest.mark.parametrize("B,H,Nb,D,block,divided", [
    (1, 1, 167, 64, 64, False), (2, 1, 115, 64, 64, False), (1, 1, 150, 64, 64, False), (1, 1, 197, 64, 64, True),
    (1, 2, 165, 64, 64, True), (1, 12, 34, 64, 64, True), (1, 3, 80, 128, 64, False), (1, 2, 105, 128, 64, True),
    (1, 4, 77, 128, 64, True), (1, 1, 102, 128, 128, True), (1, 1, 75, 128, 128, False), (1, 3, 50, 64, 128, True),
    (2, 10, 101, 64, 64, True), (1, 40, 256, 128, 128, False)])
def test_size_that_asks_for_divided_rows(lib, B, H, Nb, D, block, divided):
    from paper_2605_14513_amd.binding import HeartShape

    s = HeartShape(B, H, Nb * block, D, block)
    usual = lib.heart_attn_workspace_bytes(ctypes.byref(s))
    asks, dense = (lib.heart_attn_balanced_workspace_bytes(ctypes.byref(s), d) for d in (0, 1))
    assert (asks > usual) == divided
    assert dense in (usual, asks)


# the same on either side of the limits of rows a place (2.9; two at D = 128, block 64; 2.5 at D = block = 64 for heads of at
# most 64 blocks), of short heads beyond them, and of 4096 rows
@pytest.mark.parametrize("B,H,Nb,D,block,divided", [
    (1, 4, 371, 128, 128, True), (1, 4, 372, 128, 128, False), (1, 26, 80, 128, 128, True), (1, 16, 110, 128, 128, True),
    (1, 16, 111, 128, 128, False), (1, 4, 371, 64, 128, True), (1, 4, 372, 64, 128, True), (1, 8, 288, 64, 128, True),
    (1, 8, 289, 64, 128, False), (1, 4, 742, 64, 64, True), (1, 4, 817, 64, 64, False), (1, 40, 64, 64, 64, True),
    (1, 41, 64, 64, 64, False), (1, 41, 65, 64, 64, True), (1, 16, 128, 128, 64, True), (1, 16, 129, 128, 64, False),
    (1, 2, 846, 128, 64, True), (1, 2, 847, 128, 64, False), (1, 256, 16, 128, 128, True), (1, 257, 16, 128, 128, False),
    (1, 40, 256, 128, 64, False)])
def test_limits_of_rows_a_place(lib, B, H, Nb, D, block, divided):
    test_size_that_asks_for_divided_rows(lib, B, H, Nb, D, block, divided)


def test_product_does_not_import_the_oracle():
    pkg = os.path.join(ROOT, "paper_2605_14513_amd")
    for dirpath, _, files in os.walk(pkg):
        for f in files:
            if f.endswith((".py", ".hip", ".h")):
                text = open(os.path.join(dirpath, f)).read()
                assert "import oracle" not in text and "from oracle" not in text, f
                assert "heart_oracle" not in text, f


def test_build_knows_when_it_is_stale(lib, monkeypatch, tmp_path):
    """Every source and header counts, and the torch that the extension module was compiled against."""
    import torch

    from paper_2605_14513_amd import build as hb

    assert hb.is_built() and not hb.is_stale()
    built = min(os.path.getmtime(hb.LIB), os.path.getmtime(hb.NATIVE))
    for name in sorted(os.listdir(hb.CSRC)) + ["heart.h", "heart_diag.h"]:
        real = os.path.getmtime
        monkeypatch.setattr(os.path, "getmtime", lambda p: built + 1 if os.path.basename(p) == name else real(p))
        assert hb.is_stale(), name
        monkeypatch.undo()
    monkeypatch.setattr(torch, "__version__", "0.0.0")
    assert hb.is_stale()
    monkeypatch.undo()
    for artefact in ("LIB", "NATIVE"):
        monkeypatch.setattr(hb, artefact, str(tmp_path / "none.so"))
        assert hb.is_stale() and not hb.is_built()
        monkeypatch.undo()


def test_extension_module_has_no_thread_local_data(lib):
    """glibc (2.35) resolves every thread-local of a thread on a slow path once a library has been loaded whose own
    ones the thread never touches; libheart's error text is touched by every call."""
    import subprocess

    from paper_2605_14513_amd import build as hb

    out = subprocess.run(["readelf", "-lW", hb.NATIVE], stdout=subprocess.PIPE, check=True, text=True).stdout
    assert "LOAD" in out and "TLS" not in out
