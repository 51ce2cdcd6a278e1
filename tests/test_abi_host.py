"""Host-side checks of the C ABI (no GPU, no compute calls): the library loads, exports every symbol the
header declares, validates its arguments before touching the device, and plans launches sensibly."""
import ctypes
import os
import re

import pytest

from paper_2605_19893_amd import binding as B

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def std_params(**over):
    kw = dict(B=1, T=8, H=64, H_kv=4, d_k=192, d_v=128, l=32, d=16, l_sel=64, n_sel=16, w=512, dtype=B.SSV_BF16,
              mode=B.SSV_REFRESH, max_seq_len=32768, max_n_cmp=2047,
              k_stride=(4 * 32832 * 192, 32832 * 192, 192), v_stride=(4 * 32832 * 128, 32832 * 128, 128),
              kc_stride=(4 * 2047 * 192, 2047 * 192, 192), vc_stride=(4 * 2047 * 128, 2047 * 128, 128))
    kw.update(over)
    return B.make_params(**kw)


def test_library_exports_every_declared_symbol():
    lib = B.load_library()
    with open(os.path.join(ROOT, "include", "ssv_nsa.h")) as f:
        header = f.read()
    declared = set(re.findall(r"\b(ssv_(?:nsa|guard|tree)_[a-z_]+)\s*\(", header))
    assert declared == set(B.EXPORTS)
    for name in declared:
        assert getattr(lib, name) is not None
    assert lib.ssv_nsa_version() >= 1


def test_struct_layout_matches_header():
    # 21 four-byte fields (+ 4 bytes of padding), 18 int64 strides, 5 four-byte fields (+ padding); 18 ints and an int64 in the plan
    assert ctypes.sizeof(B.SsvNsaParams) == 22 * 4 + 18 * 8 + 6 * 4
    assert ctypes.sizeof(B.SsvNsaPlan) == 18 * 4 + 8
    with open(os.path.join(ROOT, "include", "ssv_nsa.h")) as f:
        header = f.read()
    # every field of the two structs appears in the header in the binding's order
    for struct, cls in (("ssv_nsa_params", B.SsvNsaParams), ("ssv_nsa_plan", B.SsvNsaPlan)):
        body = header[header.index("typedef struct " + struct):header.index("} " + struct + ";")]
        body = re.sub(r"/\*.*?\*/", "", body, flags=re.S)
        names = re.findall(r"\b([A-Za-z_][A-Za-z0-9_]*)\s*(?:\[\d+\])?\s*[,;]", body)
        assert names == [n for n, _ in cls._fields_], (struct, names)


def test_error_strings():
    assert B.strerror(B.SSV_OK) == "ok"
    for code in (B.SSV_EINVAL, B.SSV_EUNSUPPORTED, B.SSV_EWORKSPACE, B.SSV_ELAUNCH, B.SSV_ESTATIC):
        assert B.strerror(code) and B.strerror(code) != "unknown error"
    assert B.kernel_name(0).startswith("k_stream") and B.kernel_name(99) == ""


def test_supported_shapes():
    assert B.ssv_nsa_supported(B.SSV_BF16, 192, 128)
    assert B.ssv_nsa_supported(B.SSV_F32, 64, 64)
    assert B.ssv_nsa_supported(B.SSV_BF16, 64, 64)
    assert not B.ssv_nsa_supported(B.SSV_F32, 192, 128)


@pytest.mark.parametrize("over,code", [
    (dict(B=0), B.SSV_EINVAL), (dict(H=63), B.SSV_EINVAL), (dict(l=32, d=12), B.SSV_EINVAL),
    (dict(n_sel=2), B.SSV_EINVAL), (dict(dtype=7), B.SSV_EINVAL), (dict(mode=3), B.SSV_EINVAL),
    (dict(w=0), B.SSV_EINVAL), (dict(avg_seq_len=40000), B.SSV_EINVAL), (dict(group_size=9), B.SSV_EINVAL), (dict(scale=-1.0), B.SSV_EINVAL),
    (dict(k_stride=(1, 1, 100)), B.SSV_EINVAL), (dict(k_stride=(4 * 32832 * 192, 32832 * 192, 196)), B.SSV_EINVAL),
    (dict(mode=B.SSV_REFRESH_SHARED, group_size=9), B.SSV_EINVAL),
    (dict(exec=2), B.SSV_EINVAL), (dict(topn_home=3), B.SSV_EINVAL), (dict(max_slice_tiles=1), B.SSV_EINVAL),
    (dict(max_slice_tiles=65), B.SSV_EINVAL), (dict(imp_rows=100), B.SSV_EINVAL), (dict(exec=B.SSV_EXEC_UNFUSED, group_size=2), B.SSV_EINVAL),
    (dict(exec=B.SSV_EXEC_UNFUSED, mode=B.SSV_REFRESH_SHARED), B.SSV_EINVAL),
    (dict(q_stride=(8 * 64 * 192, 64 * 192, 100)), B.SSV_EINVAL), (dict(out_stride=(8 * 64 * 128, 64 * 128, 130)), B.SSV_EINVAL),
    # the merged schedule of 32 queries x 32 blocks does not fit the LDS next to the tiles of d_k = 192
    (dict(T=32, H=16, H_kv=4, n_sel=32, group_size=32), B.SSV_EUNSUPPORTED),
    (dict(T=129), B.SSV_EUNSUPPORTED), (dict(H=96, H_kv=4), B.SSV_EUNSUPPORTED), (dict(l_sel=128), B.SSV_EUNSUPPORTED),
    (dict(d_k=96), B.SSV_EUNSUPPORTED), (dict(n_sel=40), B.SSV_EUNSUPPORTED),
    (dict(max_seq_len=2 ** 21), B.SSV_EUNSUPPORTED),
    # rows of one (sequence, KV head) spread over 2 GiB or more: beyond the 32-bit offsets of the K loads
    (dict(max_seq_len=2 ** 19, k_stride=(4 * 2 ** 20 * 2048, 2 ** 20 * 2048, 2048)), B.SSV_EUNSUPPORTED),
    (dict(max_n_cmp=2 ** 15, kc_stride=(4 * 2 ** 15 * 2 ** 15, 2 ** 15 * 2 ** 15, 2 ** 15)), B.SSV_EUNSUPPORTED),
])
def test_bad_parameters_are_rejected_without_a_launch(over, code):
    p = std_params(**over)
    with pytest.raises(B.SsvError) as e:
        B.ssv_nsa_plan_query(p)
    assert e.value.code == code
    assert B.ssv_nsa_workspace_bytes(p) == 0
    fake = 4096   # non-null, aligned: validation of p happens before any pointer is used
    with pytest.raises(B.SsvError) as e:
        B.ssv_nsa_verify(fake, fake, fake, fake, fake, fake, fake, fake, None, None, p, fake, fake, fake, 1 << 40, 0)
    assert e.value.code == code


def test_null_misaligned_and_workspace_errors():
    p = std_params()
    need = B.ssv_nsa_workspace_bytes(p)
    assert need > 0
    a = 4096
    with pytest.raises(B.SsvError) as e:
        B.ssv_nsa_verify(None, a, a, a, a, a, a, a, None, None, p, a, a, a, need, 0)
    assert e.value.code == B.SSV_EINVAL
    with pytest.raises(B.SsvError) as e:
        B.ssv_nsa_verify(a, a + 2, a, a, a, a, a, a, None, None, p, a, a, a, need, 0)
    assert e.value.code == B.SSV_EINVAL
    for ws, nbytes in ((None, need), (a + 16, need), (a, need - 1)):
        with pytest.raises(B.SsvError) as e:
            B.ssv_nsa_verify(a, a, a, a, a, a, a, a, None, None, p, a, a, ws, nbytes, 0)
        assert e.value.code == B.SSV_EWORKSPACE


def test_plan_fills_the_chip_and_respects_limits():
    cfgs = {
        "cfg1": std_params(),
        "cfg2": std_params(B=16, T=4, max_seq_len=65536, max_n_cmp=4095),
        "cfg3": std_params(B=4, T=40, max_seq_len=131072, max_n_cmp=8191),
        "cfg4": std_params(B=32, T=16, max_seq_len=131072, max_n_cmp=8191),
    }
    for name, p in cfgs.items():
        pl = B.ssv_nsa_plan_query(p)
        H_g = p.H // p.H_kv
        assert pl.C * H_g == pl.rows_per_wg <= 64 and pl.C * pl.n_qg >= p.T
        assert pl.n_slots == pl.n_cmp_chunks + pl.n_win_splits + pl.n_slc_splits
        assert pl.n_cmp_chunks * pl.tiles_per_chunk * 64 >= p.max_n_cmp
        assert pl.max_sched_entries == pl.C * p.n_sel
        # scan launch: larger, balanced groups only where the scans keep the chip busy for several rounds; the
        # matrix-core scan (groups of up to 256 rows, one workgroup per CU) where a KV head has the rows for it
        assert pl.scan_matrix == {"cfg1": 0, "cfg2": 0, "cfg3": 1, "cfg4": 1}[name]
        assert pl.C_scan * pl.n_qg_scan >= p.T and pl.C <= pl.C_scan <= (256 if pl.scan_matrix else 128) // H_g
        assert (pl.C_scan, pl.n_qg_scan) == {"cfg1": (4, 2), "cfg2": (4, 1), "cfg3": (14, 3), "cfg4": (16, 1)}[name]
        units = p.B * p.H_kv * pl.n_qg_scan
        if pl.scan_matrix:
            wgs = units * pl.n_cmp_chunks
            # one round of one workgroup per CU, or several rounds of slices of at most 32 tiles
            assert 128 < wgs <= 256 or (wgs > 256 and pl.tiles_per_chunk <= 32), (name, wgs)
            assert pl.n_launches == (5 if name == "cfg4" else 4)
            # behind the matrix-core scan the window shares the selected-branch launch: in one round of workgroups the
            # parts of a group are cut over window tiles and schedule entries together (a slot of either branch per
            # part), in several rounds each branch has slices of its own
            assert (pl.n_win_splits, pl.n_slc_splits) == {"cfg3": (3, 3), "cfg4": (1, 2)}[name]
        else:
            wgs = units * (pl.n_cmp_chunks + pl.n_win_splits)
            # either one resident round (at most 2 workgroups per CU) or several rounds of slices of at most 32 tiles
            assert wgs >= min(256, units * ((p.max_n_cmp + 63) // 64) // 2), (name, wgs)
            assert wgs <= 512 or pl.tiles_per_chunk <= 32, (name, wgs)
        assert pl.workspace_bytes == B.ssv_nsa_workspace_bytes(p) and pl.workspace_bytes % 256 == 0
    p = std_params(group_size=2)
    pl = B.ssv_nsa_plan_query(p)
    assert (pl.C, pl.n_qg, pl.rows_per_wg) == (2, 4, 32)
    pl = B.ssv_nsa_plan_query(std_params(group_size=8))
    assert (pl.C, pl.n_qg, pl.rows_per_wg) == (8, 1, 128)
    # an explicit group size applies to both launches
    pl = B.ssv_nsa_plan_query(std_params(B=4, T=40, max_seq_len=131072, max_n_cmp=8191, group_size=2))
    assert (pl.C, pl.C_scan, pl.n_qg_scan) == (2, 2, 20)
    pl = B.ssv_nsa_plan_query(std_params(group_size=2, scan_group_size=8))
    assert (pl.C, pl.n_qg, pl.C_scan, pl.n_qg_scan) == (2, 4, 8, 1)
    pl = B.ssv_nsa_plan_query(std_params(scan_group_size=3))
    assert (pl.C, pl.n_qg, pl.C_scan, pl.n_qg_scan) == (4, 2, 3, 3)
    for bad in (-1, 9):
        with pytest.raises(B.SsvError) as e:
            B.ssv_nsa_plan_query(std_params(scan_group_size=bad))
        assert e.value.code == B.SSV_EINVAL
    # 12 queries: one group of 192 rows in the matrix-core scan; two balanced groups of 6 in the streaming kernel
    pl = B.ssv_nsa_plan_query(std_params(B=32, T=12, max_seq_len=131072, max_n_cmp=8191))
    assert (pl.C, pl.n_qg, pl.C_scan, pl.n_qg_scan, pl.scan_matrix) == (4, 3, 12, 1, 1)
    pl = B.ssv_nsa_plan_query(std_params(B=32, T=12, max_seq_len=131072, max_n_cmp=8191, scan_kernel=B.SSV_SCAN_STREAM))
    assert (pl.C, pl.n_qg, pl.C_scan, pl.n_qg_scan, pl.scan_matrix) == (4, 3, 6, 2, 0)
    # a long streaming scan of a mixed-length batch (the mean well below the maximum) starts with the work-table kernel:
    # one launch more, slots sized for the longest sequence's share of one round; a uniform batch does not
    mixed = std_params(B=32, T=8, max_seq_len=131072, max_n_cmp=8191, avg_seq_len=40000)
    pl = B.ssv_nsa_plan_query(mixed)
    pl_u = B.ssv_nsa_plan_query(std_params(B=32, T=8, max_seq_len=131072, max_n_cmp=8191))
    assert pl.scan_matrix == 0 and pl_u.scan_matrix == 0 and pl.n_launches == pl_u.n_launches + 1
    assert 2 <= pl.n_cmp_chunks <= 16 and pl.workspace_bytes == B.ssv_nsa_workspace_bytes(mixed)
    pl = B.ssv_nsa_plan_query(std_params(scan_kernel=B.SSV_SCAN_STREAM_TABLE))
    assert pl.scan_matrix == 0 and pl.n_launches == 5
    # the matrix-core scan on request: any bf16 problem of the fused execution; its groups hold up to 256 rows
    pl = B.ssv_nsa_plan_query(std_params(scan_kernel=B.SSV_SCAN_MATRIX))
    assert (pl.scan_matrix, pl.C_scan, pl.n_qg_scan, pl.n_launches) == (1, 8, 1, 4)
    pl = B.ssv_nsa_plan_query(std_params(scan_kernel=B.SSV_SCAN_MATRIX, scan_group_size=3, mode=B.SSV_REUSE))
    assert (pl.scan_matrix, pl.C_scan, pl.n_qg_scan, pl.n_launches) == (1, 3, 3, 3)
    for bad in (dict(scan_kernel=4), dict(scan_kernel=B.SSV_SCAN_STREAM_TABLE, exec=B.SSV_EXEC_UNFUSED), dict(scan_kernel=B.SSV_SCAN_MATRIX, exec=B.SSV_EXEC_UNFUSED),
                dict(scan_kernel=B.SSV_SCAN_MATRIX, dtype=B.SSV_F32, d_k=64, d_v=64), dict(scan_kernel=B.SSV_SCAN_MATRIX, scan_group_size=17)):
        with pytest.raises(B.SsvError) as e:
            B.ssv_nsa_plan_query(std_params(**bad))
        assert e.value.code == B.SSV_EINVAL, bad


def test_static_scratch_entry_point_checks_before_touching_the_device():
    fake = 4096
    big = std_params(B=16, T=4, max_seq_len=65536, max_n_cmp=4095)
    assert B.ssv_nsa_workspace_bytes(big) > B.SSV_STATIC_SCRATCH_BYTES
    with pytest.raises(B.SsvError) as e:
        B.ssv_nsa_verify_static(fake, fake, fake, fake, fake, fake, fake, fake, None, None, big, fake, fake, 0)
    assert e.value.code == B.SSV_ESTATIC and "static" in B.strerror(B.SSV_ESTATIC)
    with pytest.raises(B.SsvError) as e:      # parameter errors come first, as in the other entry points
        B.ssv_nsa_verify_static(fake, fake, fake, fake, fake, fake, fake, fake, None, None, std_params(H=63), fake, fake, 0)
    assert e.value.code == B.SSV_EINVAL
    assert 0 < B.ssv_nsa_workspace_bytes(std_params()) <= B.SSV_STATIC_SCRATCH_BYTES      # the 32K single-sequence shape fits


def test_plan_reflects_the_execution_choices():
    auto = B.ssv_nsa_plan_query(std_params())
    assert auto.topn_in_slc == 1 and auto.n_launches == 4 and auto.n_imp_chunks >= 1      # cfg1: selection inside launch B
    sep = B.ssv_nsa_plan_query(std_params(topn_home=B.SSV_TOPN_SEPARATE))
    assert sep.topn_in_slc == 0 and sep.n_launches == 5
    assert B.ssv_nsa_plan_query(std_params(B=16, T=4, max_seq_len=65536, max_n_cmp=4095)).topn_in_slc == 1   # 512 workgroups: still inside
    big = std_params(B=32, T=16, max_seq_len=131072, max_n_cmp=8191)
    assert B.ssv_nsa_plan_query(big).topn_in_slc == 0
    big.topn_home = B.SSV_TOPN_IN_SLC
    assert B.ssv_nsa_plan_query(big).topn_in_slc == 1
    reuse = B.ssv_nsa_plan_query(std_params(mode=B.SSV_REUSE))
    assert reuse.topn_in_slc == 0 and reuse.n_imp_chunks == 0 and reuse.n_launches == 2
    # several rounds of workgroups: the slice bound applies
    long_default = B.ssv_nsa_plan_query(std_params(B=32, T=16, max_seq_len=131072, max_n_cmp=8191))
    long_12 = B.ssv_nsa_plan_query(std_params(B=32, T=16, max_seq_len=131072, max_n_cmp=8191, max_slice_tiles=12))
    assert long_default.tiles_per_chunk <= 32 and long_12.tiles_per_chunk <= 12 and long_12.n_cmp_chunks > long_default.n_cmp_chunks
    # importance pass: 64 rows per workgroup for small problems, wider where a KV head has the rows and the pass is long
    assert auto.imp_rows == 64 and reuse.imp_rows == 0
    assert B.ssv_nsa_plan_query(std_params(B=4, T=40, max_seq_len=131072, max_n_cmp=8191)).imp_rows == 256
    assert B.ssv_nsa_plan_query(std_params(B=32, T=16, max_seq_len=131072, max_n_cmp=8191)).imp_rows == 256
    assert B.ssv_nsa_plan_query(std_params(B=32, T=8, max_seq_len=131072, max_n_cmp=8191)).imp_rows == 128
    assert B.ssv_nsa_plan_query(std_params(B=16, T=4, max_seq_len=65536, max_n_cmp=4095)).imp_rows == 64
    assert B.ssv_nsa_plan_query(std_params(imp_rows=256)).imp_rows == 128      # 8 queries x 16 heads fill two blocks
    assert B.ssv_nsa_plan_query(std_params(B=4, T=40, max_seq_len=131072, max_n_cmp=8191, imp_rows=64)).imp_rows == 64
    # unfused execution: every query on its own, one launch per branch plus their merges and the gate kernel
    un = B.ssv_nsa_plan_query(std_params(exec=B.SSV_EXEC_UNFUSED))
    assert (un.C, un.n_qg, un.C_scan, un.n_qg_scan, un.topn_in_slc, un.n_launches) == (1, 8, 1, 8, 0, 9)
    assert B.ssv_nsa_plan_query(std_params(exec=B.SSV_EXEC_UNFUSED, mode=B.SSV_REUSE)).n_launches == 7
    rows = 8 * 64
    assert un.workspace_bytes >= 3 * rows * 128 * 2 + un.n_slots * rows * 130 * 4


@pytest.mark.parametrize("B_,T,avg", [(32, 16, 40000), (64, 16, 40000), (16, 16, 0), (12, 16, 40000), (6, 40, 0)])
def test_explicit_slice_bound_holds_behind_the_matrix_core_scan(B_, T, avg):
    """An explicit max_slice_tiles bounds the window and selected tiles of one workgroup: launches that would otherwise take
    fewer, longer parts keep the slices the bound asks for."""
    tiles = 16 * 4 + (512 + T) // 64 + 2          # schedule entries of four queries and window tiles, at most
    for bound in (2, 5, 8, 12, 24, 32):
        pl = B.ssv_nsa_plan_query(std_params(B=B_, T=T, max_seq_len=131072, max_n_cmp=8191, avg_seq_len=avg, max_slice_tiles=bound))
        assert pl.scan_matrix == 1 and pl.max_sched_entries == 64
        groups = B_ * 4 * pl.n_qg
        if pl.n_win_splits == pl.n_slc_splits and groups * pl.n_win_splits <= 512:      # cut together in one round
            assert -(-tiles // pl.n_slc_splits) <= bound, (bound, pl.n_slc_splits)
        else:
            assert pl.n_slc_splits >= min(32, -(-64 // bound)), (bound, pl.n_slc_splits)
            assert pl.n_win_splits >= min(32, -(-(tiles - 64) // bound)), (bound, pl.n_win_splits)


@pytest.mark.parametrize("avg", [0, 40000, 127000])
@pytest.mark.parametrize("T", [16, 40, 64])
def test_walked_groups_fill_their_rounds(avg, T):
    """One workgroup per group of a mixed-length batch (it shows in the home of the selection, inside the launch up to 512
    workgroups at four queries per group) where the last round's empty places cost at most 6 tile steps; the slices stay
    what they are."""
    tiles = 64 + (512 + T) // 64 + 2
    n_qg = T // 4
    for B_ in range(256 // (4 * n_qg) + 1, 512 // (4 * n_qg) + 1):
        kw = dict(B=B_, T=T, max_seq_len=131072, max_n_cmp=8191, avg_seq_len=avg)
        pl = B.ssv_nsa_plan_query(std_params(**kw))
        groups = B_ * 4 * n_qg
        walked = avg > 0 and (512 - groups) * tiles <= 6 * 512
        assert (pl.scan_matrix, pl.C, pl.n_qg, pl.n_win_splits, pl.n_slc_splits) == (1, 4, n_qg, 1, 2)
        assert (pl.topn_in_slc, pl.n_launches) == ((1, 4) if walked else (0, 5)), (B_, groups)
        assert B.ssv_nsa_plan_query(std_params(**kw, d_k=64, d_v=64)).topn_in_slc == 0      # (three workgroups fit a CU)
        assert B.ssv_nsa_plan_query(std_params(**kw, max_slice_tiles=32)).topn_in_slc == 0
    # as few parts as one round leaves, unless they fill less than four fifths of it, would cut the schedule coarser, or three
    # workgroups fit a CU
    for B_, kw, want in ((16, {}, (2, 2)), (13, {}, (2, 2)), (12, {}, (1, 2)), (16, dict(d_k=64, d_v=64), (1, 2)), (16, dict(n_sel=24), (1, 3))):
        pl = B.ssv_nsa_plan_query(std_params(B=B_, T=16, max_seq_len=131072, max_n_cmp=8191, avg_seq_len=avg, **kw))
        assert (pl.n_win_splits, pl.n_slc_splits) == want, (kw, pl.n_win_splits, pl.n_slc_splits)


def small_params(heads, kv_heads, d, f32=False, **over):
    return std_params(**{**dict(B=1, H=heads, H_kv=kv_heads, d_k=d, d_v=min(d, 128), dtype=B.SSV_F32 if f32 else B.SSV_BF16,
                                max_n_cmp=over["max_seq_len"] // 16 - 1), **over})


@pytest.mark.parametrize("p,want", [
    # refresh: compressed and window slices of one tile up to 20 compressed tiles (fp32: 48), of two beyond
    (dict(heads=64, kv_heads=4, d=192, T=4, max_seq_len=4096), (4, 10, 32)),
    (dict(heads=16, kv_heads=1, d=192, T=4, max_seq_len=20480), (20, 10, 32)),
    (dict(heads=16, kv_heads=1, d=192, T=4, max_seq_len=21504), (11, 5, 32)),
    (dict(heads=4, kv_heads=1, d=64, f32=True, T=4, max_seq_len=49152), (48, 10, 32)),
    (dict(heads=4, kv_heads=1, d=64, f32=True, T=4, max_seq_len=50176), (25, 5, 32)),
    (dict(heads=16, kv_heads=1, d=192, T=6, max_seq_len=61440), (30, 5, 32)),
    # reuse: all branches; where the selected one has its 32 slots either way, up to 4 compressed tiles
    (dict(heads=16, kv_heads=1, d=192, T=2, max_seq_len=61440, mode=B.SSV_REUSE), (60, 10, 32)),
    (dict(heads=8, kv_heads=2, d=64, f32=True, T=3, max_seq_len=12288, mode=B.SSV_REUSE), (12, 10, 32)),
    (dict(heads=16, kv_heads=1, d=192, T=3, max_seq_len=21504, mode=B.SSV_REUSE), (11, 5, 24)),
    (dict(heads=16, kv_heads=1, d=192, T=4, max_seq_len=4096, mode=B.SSV_REUSE), (4, 10, 32)),
    (dict(heads=16, kv_heads=1, d=192, T=4, max_seq_len=5120, mode=B.SSV_REUSE), (3, 5, 32)),
    # mixed lengths: one round by the longest sequence, not by the average (7 x 2 groups of 30 + 10 tiles are more than one)
    (dict(heads=8, kv_heads=2, d=64, f32=True, T=1, B=7, max_seq_len=29889, max_n_cmp=1867, avg_seq_len=7472), (15, 5, 16)),
    (dict(heads=8, kv_heads=2, d=64, f32=True, T=1, B=7, max_seq_len=24576, max_n_cmp=1535, avg_seq_len=7472), (24, 10, 16)),
    (dict(heads=16, kv_heads=1, d=192, T=1, B=7, max_seq_len=20480, max_n_cmp=1279, avg_seq_len=7472), (20, 10, 16)),
    # the execution that the fused one replaces keeps two
    (dict(heads=16, kv_heads=1, d=192, T=2, max_seq_len=2048, exec=B.SSV_EXEC_UNFUSED), (1, 5, 8)),
])
def test_slices_of_one_tile(p, want):
    pl = B.ssv_nsa_plan_query(small_params(**p))
    assert pl.scan_matrix == 0 and (pl.n_cmp_chunks, pl.n_win_splits, pl.n_slc_splits) == want


def test_finer_cuts_do_not_cost_the_static_scratch():
    """A call whose window and selected slots fit the static array as slices of their own fits it, whatever the plan would take
    otherwise (an explicit slice bound of 32, the automatic one, asks for slices of their own)."""
    kept = 0
    for H, kv, T, n_sel, w, L in [(16, 1, 63, 24, 1024, 2048), (32, 4, 31, 24, 1024, 2048), (32, 4, 7, 32, 1024, 65536), (64, 4, 16, 16, 512, 8192)]:
        for B_ in range(1, 40):
            kw = dict(B=B_, T=T, H=H, H_kv=kv, d_k=128, d_v=128, max_seq_len=L, max_n_cmp=L // 16 - 1, n_sel=n_sel, w=w, scan_kernel=B.SSV_SCAN_MATRIX)
            own = B.ssv_nsa_plan_query(std_params(**kw, max_slice_tiles=32))
            pl = B.ssv_nsa_plan_query(std_params(**kw))
            if own.workspace_bytes <= B.SSV_STATIC_SCRATCH_BYTES:
                assert pl.workspace_bytes <= B.SSV_STATIC_SCRATCH_BYTES, kw
                # parts that one round leaves a group, and cut no coarser, would have taken more slots than there are bytes for
                groups = B_ * kv * pl.n_qg
                parts = 512 // groups
                slots = pl.n_cmp_chunks + 2 * parts
                if own.n_win_splits != own.n_slc_splits and own.n_slc_splits <= parts and parts > 1:
                    fine = slots * B_ * T * H * 130 * 4
                    assert (pl.n_win_splits == pl.n_slc_splits) or fine > B.SSV_STATIC_SCRATCH_BYTES - B_ * T * kv * (L // 16 + 64) * 4 - 4096, kw
                    kept += pl.n_win_splits != pl.n_slc_splits
    assert kept > 0


def test_plan_workspace_and_verify_agree():
    """One set of checks serves the three entry points: whatever the plan query accepts, the workspace query sizes
    and verify accepts (up to its pointer checks), and the reverse."""
    fake = 4096
    grid = [dict(), dict(T=32, H=16, H_kv=4, n_sel=32, group_size=32), dict(T=32, H=16, H_kv=4, n_sel=32, group_size=16),
            dict(T=64, H=8, H_kv=4, n_sel=32, group_size=64), dict(T=64, H=8, H_kv=4, n_sel=16, group_size=64),
            dict(d_k=64, d_v=64, T=64, H=8, H_kv=4, n_sel=32, group_size=64), dict(exec=B.SSV_EXEC_UNFUSED)]
    seen = set()
    for over in grid:
        p = std_params(**over)
        try:
            B.ssv_nsa_plan_query(p)
            plan_rc = B.SSV_OK
        except B.SsvError as e:
            plan_rc = e.code
        need = B.ssv_nsa_workspace_bytes(p)
        assert (need > 0) == (plan_rc == B.SSV_OK)
        with pytest.raises(B.SsvError) as e:      # a null query pointer: the first check after the parameters
            B.ssv_nsa_verify(None, fake, fake, fake, fake, fake, fake, fake, None, None, p, fake, fake, fake, 1 << 40, 0)
        assert e.value.code == (B.SSV_EINVAL if plan_rc == B.SSV_OK else plan_rc), over
        seen.add(plan_rc)
    assert seen == {B.SSV_OK, B.SSV_EUNSUPPORTED}


def test_shared_index_plan_keeps_the_automatic_grouping():
    p = std_params(mode=B.SSV_REFRESH_SHARED, group_size=2)
    plan = B.ssv_nsa_plan_query(p)
    auto = B.ssv_nsa_plan_query(std_params())
    assert plan.share_group == 2 and plan.C == auto.C and auto.share_group == 0
    assert B.ssv_nsa_plan_query(std_params(mode=B.SSV_REFRESH_SHARED)).share_group == auto.C
    # T = 8 queries may share one set even though a workgroup holds only 4 of them
    assert B.ssv_nsa_plan_query(std_params(mode=B.SSV_REFRESH_SHARED, group_size=8)).share_group == 8


def cmp_params(**over):
    kw = dict(B=2, H_kv=4, d_k=192, d_v=128, l=32, d=16, dtype=B.SSV_BF16, max_new_rows=8, kv_capacity=4096,
              cmp_capacity=256, k_stride=(4 * 4096 * 192, 4096 * 192, 192), v_stride=(4 * 4096 * 128, 4096 * 128, 128),
              kc_stride=(4 * 256 * 192, 256 * 192, 192), vc_stride=(4 * 256 * 128, 256 * 128, 128))
    kw.update(over)
    return B.make_cmp_params(**kw)


@pytest.mark.parametrize("over,code", [
    (dict(B=0), B.SSV_EINVAL), (dict(l=32, d=12), B.SSV_EINVAL), (dict(dtype=5), B.SSV_EINVAL),
    (dict(max_new_rows=0), B.SSV_EINVAL), (dict(cmp_capacity=0), B.SSV_EINVAL), (dict(d_k=100), B.SSV_EINVAL),
    (dict(k_stride=(1, 1, 100)), B.SSV_EINVAL), (dict(l=2048, d=16), B.SSV_EUNSUPPORTED), (dict(d_k=2048, k_stride=(4 * 4096 * 2048, 4096 * 2048, 2048), kc_stride=(4 * 256 * 2048, 256 * 2048, 2048)), B.SSV_EUNSUPPORTED),
])
def test_compress_rejects_bad_parameters_without_a_launch(over, code):
    assert ctypes.sizeof(B.SsvCmpParams) == 10 * 4 + 12 * 8
    fake = 4096
    with pytest.raises(B.SsvError) as e:
        B.ssv_nsa_compress(fake, fake, fake, fake, None, fake, fake, cmp_params(**over), 0)
    assert e.value.code == code
    with pytest.raises(B.SsvError) as e:
        B.ssv_nsa_compress(fake, fake, fake, None, None, fake, fake, cmp_params(), 0)
    assert e.value.code == B.SSV_EINVAL
