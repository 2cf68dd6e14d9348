"""CPU: the workspace of a draft that grows under one key capacity.  What pv_prepared_workspace_bytes reports for the
last pass is accepted by every pass before it, whichever of them are cut into key pieces."""
import ctypes as C

import pytest

pv = pytest.importorskip("paper_2605_04263_amd.binding")


def sizes(segments, hq, hkv, d=128):
    draft = 128 * segments
    p = pv.make_problem([512], [draft], [segments], [32], [128 * (i + 1) for i in range(segments)])
    return pv.pv_query_sizes(p, hq, hkv, d, pv.PV_BF16)


@pytest.mark.parametrize("hq,hkv", [(32, 8), (64, 8), (40, 8), (8, 8), (14, 2), (3, 3), (1024, 1024)])
def test_last_pass_holds_the_earlier_ones(hq, hkv):
    passes = [sizes(k, hq, hkv) for k in (1, 2, 5, 9, 16, 23, 31, 32, 33, 46, 64)]
    capacity = passes[-1].padded_keys
    for last in passes:
        room = pv.pv_prepared_workspace_bytes(last, capacity)
        for s in passes:
            if s.n_seg_tiles > last.n_seg_tiles:
                break
            assert pv.pv_prepared_workspace_bytes(s, capacity) <= room
            # refused for its address (looked at after the size), so that nothing is launched
            status = pv.lib.pv_prepare_kv(C.byref(s), 0x1004, 0x1000, 0x1000, None, 0, 0, s.total_tokens, capacity, 0.0,
                                          0x1000, room, None)
            assert status == pv.PV_ERR_ALIGN
