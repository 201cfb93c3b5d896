"""The rule that picks the GEMM's form for more than 64 tokens (on the host,
through qwam_probe_gemm_form).  The shapes are measured ones: where another form
took longer than the 128 x 128 tiles the rule keeps those, and the forms that
were faster stay."""

import pytest

from paper_2609_33269_amd import qwam as Q

KEPT = [
    # M, K, N, group: us of the 128 x 128 tiles, us of the form the estimate alone takes
    (920, 256, 4208, 32),     # 11.1, 15.7: one stage, 64 x 64 tiles beyond one round
    (258, 256, 11184, 32),    # 8.4, 12.7
    (1523, 256, 1008, 32),    # 7.6, 10.6: 32 x 64 tiles in their second round
    (262, 192, 11200, 32),    # 10.0, 13.7
    (473, 512, 8336, 32),     # 13.0, 18.4: two stages, more large tiles than CUs
    (4352, 128, 288, 64),     # 5.2, 5.4: one stage
    (7976, 3136, 352, 64),    # 23.3, 28.9: many tokens, few channels
    (4501, 3648, 1072, 64),   # 39.3, 45.4
    (2207, 2112, 1008, 64),   # 17.7, 19.6: the waves' ranges are whole stages (three of three, none for the fourth)
    (265, 2112, 8416, 64),    # 16.5, 18.2
]
TAKEN = [
    (415, 14336, 3072, 64, "64x64 w4"),           # 75.7, 35.7
    (100, 3072, 3072, 64, "32x64 w8"),            # 18.9, 6.2
    (333, 3072, 9216, 64, "128x128 halves"),      # 22.2, 20.6
    (333, 3072, 9216, 32, "128x128 halves"),
    (97, 256, 3312, 32, "32x64 w4"),              # 6.4, 5.0: one stage, less than a round
    (551, 256, 288, 64, "32x64 w4"),              # 6.6, 4.9
    (3258, 3136, 1072, 32, "128x128 halves"),     # 44.4, 38.0
    (4096, 3072, 14336, 64, "128x128"),
    (8192, 14336, 3072, 32, "128x128"),
    (64, 3072, 9216, 64, "few staged"),           # 19.0, 15.9 (straight to registers, through LDS)
    (33, 14336, 3072, 32, "few staged"),
    (33, 1280, 3072, 64, "few staged"),           # rows of whole lines: from three groups a wave on
    (16, 1024, 4096, 64, "few direct"),
]


@pytest.mark.parametrize("M,K,N,group", KEPT)
def test_large_tiles_are_kept_where_they_are_faster(M, K, N, group):
    assert Q.probe_gemm_form(M, N, K, group) == "128x128"


@pytest.mark.parametrize("K", [1536, 1920, 2304, 2752])
def test_two_halves_need_a_long_k_at_group_64(K):
    """208 tiles, K = 1920: 18.0 us in one piece, 19.3 in two halves."""
    assert Q.probe_gemm_form(3301, 912, K, 64) == "128x128"


@pytest.mark.parametrize("M,K,N,group,form", TAKEN)
def test_faster_forms_are_taken(M, K, N, group, form):
    assert Q.probe_gemm_form(M, N, K, group) == form


@pytest.mark.parametrize("K,form", [(1024, "few direct"), (1088, "few direct"), (1344, "few direct"), (1472, "few direct"),
                                    (1600, "few staged"), (1984, "few staged"), (2112, "few direct"), (2496, "few direct"),
                                    (2624, "few staged"), (4160, "few staged"), (1536, "few staged"), (2560, "few staged")])
def test_few_tokens_go_through_lds_where_that_is_faster(K, form):
    """Rows that are not whole lines: 2-4% slower through LDS at three groups a wave, 1-2% at five."""
    assert Q.probe_gemm_form(1, 4096, K, 64) == form and Q.probe_gemm_form(64, 16, K, 32) == form


def test_unsupported_sizes():
    for bad in ((0, 64, 64, 64), (65, 64, 64, 16), (65, 24, 64, 64), (65, 64, 100, 64)):
        with pytest.raises(Q.QwamError):
            Q.probe_gemm_form(*bad)
