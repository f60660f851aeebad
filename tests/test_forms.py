"""The rules that choose a step's forms, on the host (csrc/avs_forms.h)."""
import pytest

import forms

# Whole explicit steps on an MI355X, us, with a stage in the workgroup form and
# in the 64-lane form with 1, 2, 4 and 8 leaf shares: (dim, fp32, face, cells or
# faces, leaves, table entries, times).
MEASURED = [
    (2, 1, 0, 64, 1498, 256, (53, 81, 70, 64, 62)),
    (2, 1, 0, 144, 796, 128, (55, 66, 62, 59, 59)),
    (2, 1, 0, 12000, 100, 64, (192, 142, 153, 160, 181)),
    (2, 1, 0, 825, 94, 32, (42, 36, 38, 38, 40)),
    (2, 1, 0, 2320, 298, 128, (76, 70, 70, 69, 80)),
    (2, 0, 0, 64, 1498, 128, (58, 84, 72, 66, 64)),
    (2, 0, 0, 144, 796, 128, (50, 63, 58, 55, 54)),
    (2, 0, 0, 23584, 100, 20, (418, 327, 336, 355, 389)),
    (2, 0, 0, 2016, 100, 20, (67, 55, 57, 57, 59)),
    (2, 0, 0, 300, 100, 32, (40, 35, 37, 38, 39)),
    (3, 1, 0, 75, 1476, 80, (64, 90, 77, 70, 69)),
    (3, 1, 0, 600, 1448, 48, (100, 121, 109, 101, 100)),
    (3, 1, 0, 5760, 300, 48, (203, 168, 169, 179, 189)),
    (3, 1, 0, 2574, 748, 48, (140, 134, 129, 126, 137)),
    (3, 1, 0, 2640, 5832, 36, (449, 534, 470, 438, 447)),
    (3, 0, 0, 75, 1492, 64, (72, 98, 85, 78, 76)),
    (3, 0, 0, 504, 1184, 64, (83, 103, 92, 86, 84)),
    (3, 0, 0, 5760, 300, 48, (269, 231, 231, 243, 252)),
    (3, 0, 0, 1080, 300, 48, (89, 82, 82, 81, 83)),
    (3, 0, 0, 5760, 2472, 64, (722, 723, 695, 706, 713)),
    (2, 1, 1, 1836, 1498, 256, (73, 93, 87, 83, 82)),
    (2, 1, 1, 3050, 298, 256, (62, 67, 69, 69, 81)),
    (2, 1, 1, 14100, 100, 64, (126, 103, 112, 125, 144)),
    (2, 1, 1, 14100, 796, 64, (194, 174, 183, 196, 215)),
    (2, 1, 1, 160, 76, 20, (35, 34, 37, 37, 38)),
    (2, 0, 1, 1836, 1498, 128, (92, 112, 104, 99, 99)),
    (2, 0, 1, 1836, 298, 128, (56, 60, 60, 60, 61)),
    (2, 0, 1, 24120, 100, 32, (241, 191, 200, 215, 246)),
    (2, 0, 1, 14100, 298, 64, (193, 163, 173, 185, 204)),
    (2, 0, 1, 51400, 892, 64, (1102, 1021, 1039, 1070, 1147)),
    (3, 1, 1, 1840, 792, 64, (79, 86, 84, 82, 83)),
    (3, 1, 1, 1840, 7972, 80, (219, 313, 259, 231, 218)),
    (3, 1, 1, 17312, 300, 48, (203, 178, 187, 199, 227)),
    (3, 1, 1, 3588, 223, 40, (72, 68, 70, 70, 78)),
    (3, 1, 1, 17312, 1492, 64, (353, 345, 348, 360, 390)),
    (3, 0, 1, 1840, 1492, 64, (102, 122, 112, 108, 106)),
    (3, 0, 1, 3270, 792, 64, (116, 118, 114, 112, 120)),
    (3, 0, 1, 17312, 300, 48, (268, 236, 244, 256, 287)),
    (3, 0, 1, 7777, 792, 64, (204, 193, 191, 199, 215)),
    (3, 0, 1, 15257, 3480, 64, (838, 812, 819, 835, 865)),
]


@pytest.mark.parametrize("dim,fp32,face,count,nleaf,numax,us", MEASURED)
def test_the_chosen_form_is_near_the_fastest_measured(dim, fp32, face, count, nleaf, numax, us):
    """Alone, no slower than the best measured form by more than a tenth of the
    step, which the lanes' smaller work may cost, and 3 us (the lanes' margin)."""
    have = dict(zip((0, 1, 2, 4, 8), us))
    best = min(us)
    s = forms.shares(dim, fp32, count, nleaf, numax, face)
    if s not in have:       # between two measured counts
        a, b = max(q for q in have if q < s), min(q for q in have if q > s)
        have[s] = have[a] + (have[b] - have[a]) * (s - a) / (b - a)
    assert have[s] <= best + 3.0 + 0.1 * us[0], (s, have[s], best)


# The stages' own times of large cases, us, in the workgroup form and with 1, 2
# and 4 shares
LARGE = [
    (2, 0, 0, 32768, 298, 64, (160, 33, 50, 75)),
    (2, 0, 1, 65792, 298, 64, (180, 57, 82, 124)),
    (2, 0, 0, 32768, 1498, 128, (191, 89, 113, 149)),
    (2, 0, 1, 65792, 1498, 128, (246, 163, 191, 256)),
    (2, 1, 0, 32768, 1498, 128, (180, 85, 106, 140)),
    (2, 1, 1, 65792, 1498, 128, (198, 137, 167, 230)),
    (2, 1, 0, 32768, 1498, 256, (192, 96, 124, 176)),
    (2, 1, 1, 65792, 1498, 256, (211, 160, 205, 299)),
    (2, 1, 0, 32768, 11998, 256, (780, 572, 616, 670)),
    (2, 1, 1, 65792, 11998, 256, (778, 852, 858, 926)),
    (3, 0, 0, 25600, 468, 48, (197, 49, 67, 89)),
    (3, 0, 1, 76960, 468, 48, (248, 79, 117, 178)),
    (3, 0, 0, 25600, 5972, 64, (438, 318, 347, 336)),
    (3, 0, 1, 76960, 5972, 64, (731, 551, 592, 631)),
    (3, 1, 0, 25600, 6000, 128, (426, 332, 363, 371)),
    (3, 1, 1, 76960, 6000, 128, (599, 486, 536, 624)),
    (3, 1, 0, 25600, 18992, 128, (1191, 969, 1004, 935)),
    (3, 1, 1, 76960, 18992, 128, (1436, 1395, 1418, 1462)),
    (3, 0, 0, 36864, 468, 48, (273, 70, 83, 114)),
    (3, 0, 1, 110976, 468, 48, (352, 109, 161, 255)),
    (3, 0, 0, 36864, 5972, 64, (615, 474, 431, 447)),
    (3, 0, 1, 110976, 5972, 64, (1053, 774, 814, 937)),
    (3, 1, 0, 36864, 6000, 128, (611, 500, 460, 494)),
    (3, 1, 1, 110976, 6000, 128, (871, 689, 749, 918)),
    (3, 1, 0, 36864, 18992, 128, (1662, 1414, 1269, 1205)),
    (3, 1, 1, 110976, 18992, 128, (2013, 1911, 1958, 2066)),
]


@pytest.mark.parametrize("dim,fp32,face,count,nleaf,numax,us", LARGE)
def test_large_cases_take_a_form_near_the_fastest(dim, fp32, face, count, nleaf, numax, us):
    """Within a tenth of the stage (a step has five to eight times its time)."""
    have = dict(zip((0, 1, 2, 4), us))
    s = forms.shares(dim, fp32, count, nleaf, numax, face)
    t = have[s] if s in have else (have[2] + have[4]) / 2 if s == 3 else have[4]
    assert t <= 1.1 * min(us), (s, t, min(us))


# (dim, fp32, cells or faces, leaves, table entries, face): sizes at which a
# count chosen without regard to the other form had the lanes refused
@pytest.mark.parametrize("dim,fp32,count,nleaf,numax,face", [
    (3, 0, 75, 5200, 36, 0),
    (3, 0, 75, 5344, 36, 0),
    (2, 1, 2000, 1500, 128, 0),
    (2, 1, 4536, 1500, 128, 1),
    (2, 0, 300, 4000, 64, 0),
    (2, 0, 900, 4000, 64, 0),
    (2, 1, 3584, 1498, 256, 0),
])
def test_one_cost_ranks_the_forms_and_the_share_counts(dim, fp32, count, nleaf, numax, face):
    t = [forms.cost(dim, fp32, count, nleaf, numax, face, s) for s in range(17)]
    for most in (0, 1, 2, 3, 5, 16, 1 << 40):
        s = forms.shares(dim, fp32, count, nleaf, numax, face, most)
        assert t[s] == min(t[:2 + max(0, min(16, most) - 1)])


def test_shares_respect_every_limit():
    """Over sizes on both sides of the table and scratch limits."""
    for dim in (2, 3):
        for fp32 in (0, 1):
            for numax in (16, 36, 64, 96, 97, 128, 144, 145, 192, 193, 256, 288, 289, 512):
                for face in (0, 1):
                    for count in (1, 64, 65, 700, 4536, 16384, 16385, 110976):
                        for nleaf in (1, 64, 300, 1500, 2200, 5200, 19972):
                            for most in (0, 1, 2, 5, 1 << 40):
                                s = forms.shares(dim, fp32, count, nleaf, numax, face, most)
                                assert 0 <= s <= min(max(1, most), 16)
                                assert s == 0 or forms.form(dim, fp32, numax)


# Whole explicit steps, us, with four waves per cell in pass C and with one:
# (dim, fp32, cells, leaves, table entries, four, one)
PASSC = [
    (2, 1, 64, 1530, 120, 54, 69),
    (2, 1, 64, 1198, 128, 50, 62),
    (2, 1, 144, 795, 120, 47, 55),
    (2, 1, 12000, 76, 32, 125, 102),
    (2, 1, 7000, 148, 32, 86, 74),
    (2, 1, 7000, 507, 72, 125, 114),
    (2, 0, 64, 1200, 72, 54, 69),
    (2, 0, 144, 796, 64, 50, 58),
    (2, 0, 64, 300, 72, 40, 44),
    (2, 0, 12000, 76, 32, 181, 136),
    (2, 0, 3584, 76, 64, 72, 59),
    (2, 0, 7000, 298, 64, 155, 135),
    (3, 1, 75, 1513, 72, 64, 86),
    (3, 1, 75, 1184, 64, 61, 77),
    (3, 1, 1080, 1492, 64, 105, 126),
    (3, 1, 5760, 64, 16, 120, 104),
    (3, 1, 2574, 288, 16, 86, 82),
    (3, 0, 75, 1532, 24, 72, 96),
    (3, 0, 75, 468, 48, 52, 61),
    (3, 0, 288, 300, 24, 51, 54),
    (3, 0, 5760, 64, 16, 159, 139),
    (3, 0, 2574, 288, 16, 113, 109),
]


@pytest.mark.parametrize("dim,fp32,nc,nleaf,numax,four,one", PASSC)
def test_pass_c_takes_the_faster_measured_form(dim, fp32, nc, nleaf, numax, four, one):
    """By more than the 1 us and 2 % that two runs may differ by."""
    us = one if forms.wave(dim, fp32, nc, nleaf, numax) else four
    assert us <= min(four, one) + 1.0 + 0.02 * four


def test_the_gpu_tests_sizes_are_in_the_forms_they_are_for():
    import test_gpu_forms as G
    for name, prec in G.ALONE + [(n, prec) for names, prec in G.BATCHED for n in names]:
        G.build(name, prec)
