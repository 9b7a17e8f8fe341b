"""Launch shapes chosen by token count: every family's entry covers its row at every supported width for short
launches too, and the backward that keeps its slots in a static array finds a plan that fits wherever the plan of
lnmod_backward does not."""
import os

import pytest

from paper_2605_17923_amd import lnmod, lnmod_tools as T


@pytest.mark.parametrize("tokens", [1, 300, 2500, 20000, 400000])
def test_every_entry_covers_its_row_whatever_the_token_count(tokens):
    for fam in range(T.LNMOD_FAMILIES):
        for dtype, vec in ((0, 8), (1, 4)):
            for D in range(8, 8193, 8):
                st, (K, VPL, R, per_cu) = T.lnmod_table_shape(fam, D, dtype, tokens)
                assert st == 0 and K * VPL * 64 >= D // vec, (fam, dtype, D)
                assert R in (1, 2) and 1 <= per_cu and K * per_cu <= 32, (fam, dtype, D)


@pytest.mark.parametrize("B,S,D,dtype,rc", [(471, 127, 3824, 1, 1), (17, 5276, 5768, 0, 1), (188, 352, 3840, 0, 1),
                                            (146, 348, 3832, 1, 1), (419, 165, 3936, 1, 0), (1936, 297, 1592, 1, 0),
                                            (1428, 638, 1544, 0, 0), (123, 4572, 1080, 0, 1), (1051, 56, 3984, 1, 1)])
def test_static_backward_takes_problems_whose_usual_plan_needs_more(B, S, D, dtype, rc):
    # these were within the array before their launch shapes got more blocks; without a GPU an accepted call
    # ends at the first HIP call (LNMOD_ELAUNCH), a refused one before it
    if os.path.exists("/dev/kfd"):
        pytest.skip("the addresses are made up: only for a host without a GPU")
    A = 16
    st = lnmod.lnmod_backward_static(A, A, None, A, B, S, D, 1e-6, None, None if rc else A, None if rc else A, A, A, A,
                                     dtype, lnmod.LNMOD_PER_SAMPLE)
    assert st == lnmod.LNMOD_ELAUNCH


def test_one_samples_workspace_never_shrinks_as_its_rows_grow():
    # a caller sizes its workspace for the longest clip and passes it for shorter ones
    queries = (lambda T, D: lnmod.lnmod_backward_workspace_bytes(1, T, D, lnmod.LNMOD_PER_SAMPLE),
               lambda T, D: lnmod.lnmod_gated_backward_workspace_bytes(1, T, D),
               lambda T, D: lnmod.lnmod_qknorm_backward_workspace_bytes(T, D))
    for D in range(8, 8193, 8):
        rows = [1, 2, 100, 255, 256, 257, 511, 512, 513, 767, 1024, 1025, 2048, 4096, 75600, 400000]
        rows += [72000000 // (16 * n) + k for n in (D // 8, D // 4) for k in (-1, 0, 1, 2)]    # short | long launches
        rows = sorted(t for t in set(rows) if t > 0)
        for q in queries:
            sizes = [q(t, D) for t in rows]
            assert sizes == sorted(sizes) and sizes[0] > 0, (D, rows, sizes)


# (family, D, dtype, rows, (waves, chunks per lane, rows per step, blocks per CU)): both sides of the lines where a width
# below the one that its table entry was timed at, another alignment or another size wants another shape
@pytest.mark.parametrize("family,D,dtype,rows,shape", [
    # per token: rows that are not whole lines, beyond short launches, from D = 3336 on
    (T.LNMOD_FAMILY_TOKEN_BACKWARD_NO_DSHIFT, 3704, 0, 40000, (4, 2, 2, 2)),
    (T.LNMOD_FAMILY_TOKEN_BACKWARD_NO_DSHIFT, 3704, 0, 5000, (8, 1, 1, 2)),
    (T.LNMOD_FAMILY_TOKEN_BACKWARD, 4008, 0, 5000, (8, 1, 1, 1)),
    (T.LNMOD_FAMILY_TOKEN_BACKWARD, 3208, 0, 40000, (8, 1, 1, 2)),
    (T.LNMOD_FAMILY_TOKEN_BACKWARD, 3400, 0, 40000, (4, 2, 1, 2)),
    # short forward, D = 5128 ... 5376: two blocks of one row whatever the alignment
    (T.LNMOD_FAMILY_FORWARD, 5376, 0, 3044, (4, 3, 1, 2)),
    (T.LNMOD_FAMILY_FORWARD, 5272, 0, 3044, (4, 3, 1, 2)),
    # backward, D = 264 ... 504, and its fp32 form at D = 3076 ... 3328
    (T.LNMOD_FAMILY_BACKWARD, 264, 0, 200000, (1, 1, 2, 8)),
    (T.LNMOD_FAMILY_BACKWARD, 504, 0, 60000, (1, 1, 2, 8)),
    (T.LNMOD_FAMILY_BACKWARD, 440, 0, 30000, (1, 1, 2, 4)),
    (T.LNMOD_FAMILY_BACKWARD, 512, 0, 200000, (1, 1, 1, 8)),
    (T.LNMOD_FAMILY_BACKWARD_RECOMPUTE, 312, 0, 400000, (1, 1, 2, 8)),
    (T.LNMOD_FAMILY_BACKWARD, 3116, 1, 15000, (5, 4, 2, 1)),
    # forward, D = 1288 ... 1528 and 2568 ... 2808
    (T.LNMOD_FAMILY_FORWARD, 1408, 0, 60000, (1, 3, 1, 8)),
    (T.LNMOD_FAMILY_FORWARD, 1400, 0, 60000, (1, 3, 2, 4)),
    (T.LNMOD_FAMILY_FORWARD, 1288, 0, 40000, (1, 3, 1, 8)),
    (T.LNMOD_FAMILY_FORWARD, 1288, 0, 100000, (1, 3, 2, 4)),
    (T.LNMOD_FAMILY_FORWARD, 2568, 0, 40000, (2, 3, 1, 4)),
    (T.LNMOD_FAMILY_FORWARD, 2680, 0, 40000, (4, 2, 1, 3)),
    # gated forward
    (T.LNMOD_FAMILY_GATED_FORWARD, 5632, 0, 700, (4, 3, 1, 2)),
    (T.LNMOD_FAMILY_GATED_FORWARD, 5048, 0, 7131, (4, 3, 1, 1)),
    (T.LNMOD_FAMILY_GATED_FORWARD, 2568, 0, 14000, (4, 2, 1, 3)),
    (T.LNMOD_FAMILY_GATED_FORWARD, 1144, 0, 37000, (2, 2, 1, 4)),
    (T.LNMOD_FAMILY_GATED_FORWARD, 1144, 0, 90000, (2, 2, 1, 3)),
    (T.LNMOD_FAMILY_GATED_FORWARD, 3116, 1, 15000, (4, 4, 2, 1)),
    (T.LNMOD_FAMILY_GATED_FORWARD, 7168, 1, 488, (8, 4, 2, 1)),
    (T.LNMOD_FAMILY_GATED_FORWARD, 7168, 1, 256, (8, 4, 1, 1)),
    (T.LNMOD_FAMILY_GATED_FORWARD, 8192, 1, 1983, (8, 4, 2, 2)),
    (T.LNMOD_FAMILY_GATED_FORWARD, 1024, 1, 2441, (1, 4, 2, 4)),
    (T.LNMOD_FAMILY_GATED_FORWARD, 4612, 1, 1354, (5, 4, 2, 1)),
    # query / key normalisation
    (T.LNMOD_FAMILY_QKNORM_FORWARD, 5128, 0, 6142, (6, 2, 2, 1)),
    (T.LNMOD_FAMILY_QKNORM_FORWARD, 3136, 0, 9885, (5, 2, 2, 3)),
    (T.LNMOD_FAMILY_QKNORM_FORWARD, 8192, 0, 1100, (8, 2, 2, 1)),
    (T.LNMOD_FAMILY_QKNORM_BACKWARD, 1920, 0, 45000, (2, 2, 2, 3)),
    (T.LNMOD_FAMILY_QKNORM_BACKWARD, 2048, 0, 45000, (2, 2, 2, 2)),
    (T.LNMOD_FAMILY_QKNORM_BACKWARD, 3160, 0, 27000, (4, 2, 2, 2)),
    (T.LNMOD_FAMILY_QKNORM_BACKWARD, 3200, 0, 27000, (4, 2, 2, 1)),
])
def test_shapes_on_both_sides_of_a_line(family, D, dtype, rows, shape):
    assert T.lnmod_table_shape(family, D, dtype, rows) == (0, shape)


@pytest.mark.parametrize("D,rows,segments,kernel,blocks", [
    (512, 150000, 300, "1, 1, 2", 4096),          # the short table's entry with its two rows per step
    (768, 150000, 300, "2, 1, 2", 4096),
    (1024, 60000, 300, "2, 1, 1", 3072),          # one row per step ...
    (1024, 150000, 300, "2, 1, 2", 1024),         # ... but the long table's on large launches of longer segments
    (1024, 150000, 600, "2, 1, 1", 3072),
    (1280, 60000, 300, "3, 1, 1", 2048),          # the long table's, except on very short segments
    (1280, 60000, 600, "3, 1, 1", 3072),
    (1408, 60000, 120, "3, 1, 1", 2048),
    (1536, 52000, 96, "3, 1, 1", 2048),
    (1536, 120000, 150, "3, 1, 2", 1024),         # the long table's on large launches
    (5376, 2843, 20, "3, 4, 2", 1422)])           # (1422 steps for six blocks per CU)
def test_forward_on_many_short_segments_takes_the_shape_of_its_size(D, rows, segments, kernel, blocks):
    text = T.lnmod_describe_launch(0, None, segments, rows, True, D, 0, lnmod.LNMOD_PER_SAMPLE)
    assert text.startswith("fwd_split_kernel<bf16_io, %s, " % kernel) and ", 4, true>" in text, text
    assert abs(int(text.split("grid=")[1].split()[0]) - blocks) <= 32, text
