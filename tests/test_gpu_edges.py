"""Edges of the selection inside the selected-branch launch (groups of 64 blocks, 512 or 1024 blocks in flight, the
remainder, ties) and of the matrix-core scan's two half-phases (slices of one to five tiles, a last tile of one row, no
tile at all), against the oracle and against the selection's own launch, whose kernel is another one."""
import numpy as np
import pytest

import ssv_inputs as si
from parity import check, compare
from test_gpu_parity import dev_mod, run_refresh  # noqa: F401  (fixture)

pytestmark = pytest.mark.gpu


def select_both_ways(dev_mod, oracle, case):
    """The sets of the selection inside the selected-branch launch and of its own launch; the plan says that each is what ran
    (importances that do not fit that launch's tile buffers are selected from in the launch of their own whatever the caller asks)."""
    from paper_2605_19893_amd import binding as B
    dev, _, _, inside = run_refresh(dev_mod, oracle, case, topn_home=B.SSV_TOPN_IN_SLC)
    assert dev.plan.topn_in_slc == 1
    dev, _, _, own = run_refresh(dev_mod, oracle, case, topn_home=B.SSV_TOPN_SEPARATE)
    assert dev.plan.topn_in_slc == 0
    return inside, own


@pytest.mark.parametrize("blocks,d_k", [(n, d) for n in (1, 63, 64, 65, 66, 128, 130, 512, 513, 577, 1024, 1027, 1089, 2050) for d in (64, 192)
                                        if (n, d) != (2050, 64)])       # (that many importances do not fit at d_k = 64)
def test_selection_at_the_edges_of_its_groups(dev_mod, oracle, blocks, d_k):  # noqa: F811
    d_v = 64 if d_k == 64 else 128
    case = si.make_case(f"sel_edge_{blocks}_{d_k}", "bf16", 1, 3, 16, 1, d_k, d_v, si.STD_NSA, [blocks * 64 - 1], 301 + blocks, rho=0.3)
    inside, own = select_both_ways(dev_mod, oracle, case)
    assert np.array_equal(inside, own)


@pytest.mark.parametrize("n_cmp", [0, 3, 255, 300, 3000])
@pytest.mark.parametrize("n_init", [0, 1, 4])
def test_selection_with_few_compressed_rows_is_one_of_ties(dev_mod, oracle, n_cmp, n_init):  # noqa: F811
    """Blocks without a compressed row have importance 0: many candidates of the same value, the smaller indices win."""
    nsa = si.NsaParams(l=32, d=16, l_sel=64, n_sel=16, w=512, n_init=n_init, n_local=2)
    case = si.make_case(f"sel_ties_{n_cmp}_{n_init}", "f32", 1, 2, 4, 1, 64, 64, nsa, [70000], 401 + n_cmp)
    case.n_cmp[:] = n_cmp
    inside, own = select_both_ways(dev_mod, oracle, case)
    assert np.array_equal(inside, own)


def takes_balanced_split(plan, max_n_cmp):
    """Even slices of ntc tiles are ceil(ntc / slices) tiles each and none is superfluous; ranges of the balanced split cover the
    longest sequence and its fixed cost with one slot to spare."""
    return (plan.n_cmp_chunks - 1) * plan.tiles_per_chunk >= max(1, -(-max_n_cmp // 64))


@pytest.mark.parametrize("T", [12, 17])
@pytest.mark.parametrize("rows", [0, 1, 63, 64, 65, 128, 129, 193, 257, 320])
def test_matrix_scan_of_few_tiles(dev_mod, oracle, rows, T):  # noqa: F811
    """Even slices (of one sequence, of three); ranges of the balanced split that hold one tile each; and (one query per workgroup of the scan: fewer, longer
    ranges) ranges that hold all tiles of one pair and go on into the next, with the same sequence's metadata and with another's."""
    from paper_2605_19893_amd import binding as B
    length = 32 + 16 * (rows - 1) if rows else 20
    long = length + 1100
    for name, lens, H_kv, avg, scan_group in (("even", [length], 1, 0, 0), ("even_batch", [length, 900, length], 1, 0, 0),
                                              ("short_ranges", [length, long, length], 1, 1, 0),
                                              ("long_ranges", 4 * [length, long, length], 2, 1, 1)):
        case = si.make_case(f"scan_edge_{name}_{rows}_{T}", "bf16", len(lens), T, 16 * H_kv, H_kv, 192, 128, si.STD_NSA, lens, 501 + rows, rho=0.5,
                            cmp_over_drafts=False)
        assert int(case.n_cmp[0]) == rows
        dev = dev_mod.DeviceCase(case, scan_kernel=B.SSV_SCAN_MATRIX, avg_seq_len=avg)
        dev.set_group_size(0, B.SSV_REFRESH, scan_group_size=scan_group)
        plan = dev.plan
        assert plan.scan_matrix == 1 and takes_balanced_split(plan, int(case.n_cmp.max())) == name.endswith("ranges")
        if name == "long_ranges":       # more pairs than ranges: some range holds more than one
            assert len(lens) * H_kv > 256 // plan.n_qg_scan
        print(f"[run] {case.name} plan={plan.as_dict()}", flush=True)
        dev.run()
        out, sel = dev.results()
        check(case, compare(case, oracle, oracle.nsa_verify(case), out, sel))
