"""Where a prefill call is split over its key tiles (jf_prefill_workspace_bytes
is 0 where row blocks stay whole).  CPU only: the plan takes 256 compute units
where there is no device."""
import pytest

from paper_2609_17475_amd import jfkv


def splits(hq, hkv, d, group, T, prefix):
    lay = jfkv.layout(256, hkv, d, group, 4000)
    return jfkv.jf_prefill_workspace_bytes(lay, T, hq, prefix) > 0


@pytest.mark.parametrize("hq,hkv,d,group,T,prefix", [
    # measured (us, split against whole): the row blocks of a chunk without a
    # prefix are short, and a share that touches many pays for each
    (64, 8, 128, 64, 1194, 0),    # 89.9 / 67.6
    (64, 8, 128, 64, 2509, 0),    # 255.7 / 183.2
    (64, 8, 128, 64, 7424, 0),    # 1502 / 1134
    (40, 8, 128, 64, 2174, 0),    # 130.6 / 113.3
    (40, 8, 128, 64, 4751, 0),    # 421.6 / 353.8
    (32, 8, 128, 64, 2097, 0),    # 103.4 / 92.5
    (32, 8, 128, 32, 4096, 0),    # 259.3 / 230.0
    (32, 8, 128, 64, 7917, 0),    # 779.5 / 704.1
    (16, 2, 64, 32, 5981, 0),     # 214.1 / 174.3
    (64, 8, 128, 64, 1792, 53),   # 182.2 / 157.5
    # two full turns over a long prefix: too little to gain for 71 MB of scratch
    (32, 8, 128, 64, 2048, 32768),    # 1,647 / 1,669
    (32, 8, 128, 64, 2048, 65536),    # 3,189 / 3,206
    (32, 8, 128, 64, 2048, 131072),   # 6,291 / 6,283
])
def test_whole_row_blocks_where_a_split_costs_more(hq, hkv, d, group, T, prefix):
    assert not splits(hq, hkv, d, group, T, prefix)


@pytest.mark.parametrize("hq,hkv,d,group,T,prefix", [
    (24, 4, 256, 64, 256, 196608),   # 2,504 / 13,494
    (32, 8, 128, 64, 1000, 7000),    # 217 / 395
    (4, 1, 128, 64, 5786, 0),        # 97.1 / 201.0
    (4, 1, 128, 64, 100, 500),       # 17.8 / 38.7
    (16, 2, 64, 32, 2048, 32768),    # 556 / 1,094
    (32, 8, 128, 64, 3072, 32768),   # 2,531 / 3,394
    (32, 8, 128, 64, 2048, 16384),   # 874 / 897
    (32, 8, 128, 64, 2048, 64),      # 120 / 130
    (40, 8, 128, 64, 2048, 86),      # 141 / 161
    (24, 4, 256, 64, 1792, 216),     # 163 / 189
    (24, 4, 256, 64, 2048, 8192),    # 995 / 1,299
])
def test_split_where_it_pays(hq, hkv, d, group, T, prefix):
    assert splits(hq, hkv, d, group, T, prefix)


@pytest.mark.parametrize("hq,hkv,d", [(32, 8, 128), (4, 1, 128), (24, 4, 256), (16, 2, 64), (8, 8, 64),
                                      (64, 1, 128), (128, 1, 256), (96, 1, 64), (512, 1, 256)])
def test_sizes_the_python_entry_does_not_ask_about_are_whole(hq, hkv, d):
    """The Python entry points spare the smallest calls the question."""
    asked = [(T, p) for p in (0, 1, 17, 40, 63) for T in range(1, 257)
             if not jfkv._prefill_scratch_bytes(jfkv.layout(256, hkv, d, 64, 4000), T, hq, p)]
    assert (64, 0) in asked and (1, 63) in asked
    assert not any(splits(hq, hkv, d, 64, T, p) for T, p in asked)


@pytest.mark.parametrize("T,prefix", [(273, 19), (276, 3), (269, 21)])
def test_shares_across_row_blocks_are_counted(T, prefix):
    """Sixteen shares of five row blocks of two to six tiles: some begin in one row
    block and end in the next (32 us against 27 with whole row blocks)."""
    assert not splits(32, 8, 128, 64, T, prefix)
