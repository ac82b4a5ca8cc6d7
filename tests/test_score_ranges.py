"""How the scoring passes share out their work, on the CPU: the functions that the launches themselves call, through the test hook."""
import pytest

from paper_2507_13681_amd import binding


@pytest.mark.parametrize("B,Hq,Hkv,n,w,mode", [
    (1, 32, 8, 32768, 64, 0), (4, 64, 8, 16384, 64, 0), (1, 32, 8, 131072, 256, 1), (2, 12, 4, 50001, 97, 3),
    (4, 64, 8, 16384, 16, 2), (1, 8, 1, 262144, 256, 2), (3, 64, 8, 4000, 16, 2),
    # one KV head and a window: ls_score takes as many keys as an int counts, and 768 ranges times 2^23 blocks are more than 2^32
    (1, 3, 1, 715827968, 32, 0), (1, 4, 1, 800000001, 64, 0), (1, 4, 1, 2147483000, 64, 0), (1, 1, 1, 2147483000, 128, 0), (1, 8, 1, 1500000063, 256, 1)])
def test_every_key_lies_in_one_range(B, Hq, Hkv, n, w, mode):
    route = binding.score_route(binding.make_shape(B, Hq, Hkv, 64, n, 1, w, "bf16"), mode)
    ranges, begins, unit = route["ranges"], route["begins"], 64 if mode == 2 else 128
    units = -(-n // unit)
    assert ranges > 1
    assert begins == [min(n, units * x // ranges * unit) for x in range(ranges + 1)]       # in whole numbers of any size
    assert begins[0] == 0 and begins[-1] == n and all(a < b for a, b in zip(begins, begins[1:]))


@pytest.mark.parametrize("Hq,Hkv,n,w,d", [(4, 1, 262144, 16, 128), (8, 1, 131072, 32, 64), (8, 2, 262144, 16, 128), (16, 4, 131072, 32, 64), (3, 3, 262144, 31, 128)])
def test_long_caches_of_few_heads_have_work_for_every_unit(Hq, Hkv, n, w, d):
    """Retention: ranges enough for two workgroups on each of 256 compute units, or 256 of one head."""
    route = binding.score_route(binding.make_shape(1, Hq, Hkv, d, n, 1, w, "bf16"), 2)
    assert route["ranges"] * Hkv >= min(510, 256 * Hkv)


@pytest.mark.parametrize("B,Hq,Hkv,n,w,d,heads,rows,shares", [
    (4, 64, 8, 16384, 64, 64, 5, 32, 2), (4, 64, 8, 16384, 64, 128, 5, 32, 2),     # 640 workgroups of eight chunks, 1280 of four
    (1, 32, 8, 131072, 128, 128, 1, 32, 1), (1, 32, 8, 32768, 64, 128, 2, 64, 2),  # two each with more than 1024
    (1, 16, 4, 5003, 48, 64, 4, 48, 4)])
def test_bands_are_shared_out_by_their_own_chunks(B, Hq, Hkv, n, w, d, heads, rows, shares):
    """Explicit positions: a second round of workgroups where they keep four chunks of the band, not of the window."""
    route = binding.score_route(binding.make_shape(B, Hq, Hkv, d, n, 1, w, "bf16"), 1, True)
    assert (route["band_heads"], route["band_rows"], route["band_shares"]) == (heads, rows, shares)


@pytest.mark.parametrize("B,Hq,Hkv,n,w,d,cut", [
    (4, 64, 8, 16384, 64, 128, False), (8, 64, 8, 8192, 64, 128, False), (1, 32, 8, 32768, 64, 128, True), (1, 64, 8, 32768, 64, 128, True), (1, 32, 8, 131072, 256, 128, True), (4, 32, 8, 16384, 64, 128, True), (4, 64, 8, 3000, 64, 128, True),
    (4, 64, 8, 16384, 64, 64, False), (1, 32, 8, 32768, 64, 64, False), (1, 16, 4, 131072, 64, 64, False)])
def test_explicit_positions_have_no_few_long_ranges(B, Hq, Hkv, n, w, d, cut):
    """Rows at explicit positions see parts of the context: a few long ranges come out uneven, and at d = 64 any gain nothing.  The newest rows of the same shapes are cut."""
    shape, mode = binding.make_shape(B, Hq, Hkv, d, n, 1, w, "bf16"), 0 if w <= 128 else 1
    ranges = binding.score_route(shape, 1, True)["ranges"]
    assert (ranges >= 16 or -(-n // 128) < 8 * ranges) if cut else ranges == 0
    assert binding.score_route(shape, mode)["ranges"] > 0 and binding.score_route(shape, 3, True)["ranges"] == ranges
