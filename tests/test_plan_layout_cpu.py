"""The planner's choice of layout and split for batches that leave both to it (CPU only): whatever
it chooses is one of the partitions that can be asked for by name, so it is covered by what those
are tested for; any option given turns the choice off."""
import numpy as np
import pytest

from paper_2604_16395_amd import plan_opts, s2l_plan_host
from tests.test_plan_cpu import _coverage

LAYOUTS = [(256, 1), (128, 1), (128, 2)]


def _same(a, b):
    return a[0].num_items == b[0].num_items and a[0].workspace_bytes == b[0].workspace_bytes and np.array_equal(a[1], b[1])


@pytest.mark.parametrize("seed", range(40))
def test_choice_is_a_partition_that_can_be_asked_for(seed):
    rng = np.random.default_rng(seed)
    R = int(rng.integers(1, 20))
    P = rng.integers(0, int(rng.choice([1, 300, 3000, 30000])), size=R).astype(np.int32)
    C = rng.integers(0, int(rng.choice([40, 300, 1500])), size=R).astype(np.int32)
    C[0] = 50
    hq, hkv = [(8, 2), (32, 8), (64, 8), (8, 1), (6, 2), (4, 4)][seed % 6]
    auto = s2l_plan_host(P, C, hq, hkv, with_items=True)
    info = auto[0]
    assert (info.tile_cols, info.key_halves) in LAYOUTS
    asked = [s2l_plan_host(P, C, hq, hkv, plan_opts(tile_cols=info.tile_cols, key_halves=info.key_halves, target_items=t),
                           with_items=True) for t in (0, 1)]
    assert any(_same(auto, x) for x in asked)
    _coverage(P, C, hq, hkv, auto[1][auto[1][:, 0] >= 0], info.tile_cols)
    # an option of any kind: the fixed rules
    for o in (plan_opts(target_items=256), plan_opts(min_split_keys=512), plan_opts(max_splits=16)):
        fixed, _ = s2l_plan_host(P, C, hq, hkv, o)
        assert fixed.tile_cols == 256 or fixed.key_halves == 2


def test_choice_on_short_and_long_ranges():
    # one chunk without a prefix: 128-column tiles in one round, no merge
    info, _ = s2l_plan_host([0], [512], 32, 8)
    assert info.tile_cols == 128 and info.num_split_reqs == 0
    # a long range behind few columns: narrower tiles, two workgroups a CU
    info, _ = s2l_plan_host([20000], [100], 8, 1)
    assert info.tile_cols == 128
    # long ranges that fill the GPU: 256 columns
    for P, C in (([8192], [512]), ([32768] * 8, [512] * 8)):
        info, _ = s2l_plan_host(P, C, 32, 8)
        assert info.tile_cols == 256


@pytest.mark.parametrize("P,one_round", [([5000 * (i + 1) for i in range(6)], True), ([16000] * 24, False), ([2047], True)])
def test_decode_rows_keep_one_round_unless_its_pieces_are_long(P, one_round):
    """Decode pieces are cut to 4096 keys only where one round of workgroups would leave them at 8192
    keys or more; else the batch stays within one round."""
    info, _ = s2l_plan_host(P, [1] * len(P), 32, 8)
    assert info.tile_cols == 16 and info.num_split_reqs > 0
    assert (info.num_items <= 256) == one_round
    assert info.split_keys <= (8192 if one_round else 4096)


@pytest.mark.parametrize("P,hq,hkv,cut", [([75125] * 46, 8, 1, False), ([60000] * 25, 64, 8, False),
                                          ([40000, 30000] + [3000] * 28, 32, 8, True), ([16000] * 24, 32, 8, True)])
def test_decode_pieces_are_cut_only_where_the_items_end_earlier(P, hq, hkv, cut):
    """One round of workgroups that is nearly full of equal items (230 of 15026 keys, 200 of 60001)
    has nothing to gain from a cut to 4096 keys, whose last round is partly filled; one that a few
    long requests dominate, or that leaves a quarter of the workgroups idle, has."""
    info, _ = s2l_plan_host(P, [1] * len(P), hq, hkv)
    one, _ = s2l_plan_host(P, [1] * len(P), hq, hkv, plan_opts(target_items=256))
    assert one.num_items <= 256 and one.split_keys >= 8192
    assert info.split_keys == (4096 if cut else one.split_keys)


@pytest.mark.parametrize("P,C,hq,hkv", [([0], [1456], 28, 4), ([2663] * 2, [627] * 2, 28, 4), ([4528] * 3, [262] * 3, 32, 8),
                                        ([0] * 2, [471] * 2, 64, 1), ([22635], [532], 64, 1)])
def test_choice_is_one_that_e4m3_pages_bear(P, C, hq, hkv):
    """Batches whose narrower layouts gain little over bf16 pages and lose over e4m3 ones (measured:
    6 to 28% there, with plain or quantised queries) keep the default, as the plan serves both."""
    info, _ = s2l_plan_host(P, C, hq, hkv)
    assert info.tile_cols == 256


@pytest.mark.parametrize("P,split", [([299] * 8, False), ([511, 40], False), ([512], True), ([300, 700], True)])
def test_short_decode_rows_are_left_whole(P, split):
    """Up to 512 keys the merge costs more than two pieces save, unless the caller asks for pieces."""
    info, _ = s2l_plan_host(P, [1] * len(P), 32, 8)
    assert info.tile_cols == 16 and (info.num_split_reqs > 0) == split
    info, _ = s2l_plan_host(P, [1] * len(P), 32, 8, plan_opts(min_split_keys=256))
    assert info.num_split_reqs > 0
