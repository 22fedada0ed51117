"""Which form of the projection kernel a tensor takes: the forms that were measured to be ahead, on the CPU."""
import os

import pytest

from paper_1905_10830_amd import binding as fmtc
from paper_1905_10830_amd.synth import NCHW, NHWC


@pytest.fixture(scope="module", autouse=True)
def library():
    if not os.path.exists(fmtc.LIB_PATH):
        from paper_1905_10830_amd import build

        build.build()
    return fmtc.load_library()


def form(C, P, layout, bits, keep=None):
    shape = (1, 1, P, C) if layout == NHWC else (1, C, 1, P)
    return fmtc.test_projection(shape, layout, bits, keep).split(" nhwc" if layout == NHWC else " nchw")[0]


# us of the kernel in the form named and in the other of the two, as measured
@pytest.mark.parametrize("C,P,layout,bits,want,ahead,behind", [
    (1000, 1024, NHWC, 8, "wide", 48, 67), (1000, 1024, NHWC, 6, "split 1x4", 42, 44), (1000, 4096, NHWC, 3, "wide", 59, 78),
    (1000, 4096, NHWC, 6, "wide", 70, 94), (1000, 5184, NHWC, 6, "split 1x4", 115, 125), (1000, 20000, NHWC, 6, "wide", 305, 369),
    (500, 8192, NHWC, 6, "wide", 38, 51), (500, 10400, NHWC, 6, "split 1x4", 61, 67), (500, 40000, NHWC, 8, "wide", 189, 236), (1000, 6496, NHWC, 7, "wide", 132, 161), (580, 18496, NHWC, 6, "split 1x4", 115, 147),
    (644, 13696, NHWC, 7, "wide", 132, 151), (570, 11552, NCHW, 6, "split 1x4", 94, 113),
    (404, 16000, NHWC, 6, "wide", 55, 66), (300, 28800, NHWC, 8, "split 1x4", 77, 106), (300, 28800, NHWC, 6, "split 1x4", 66, 74),
    (1001, 8992, NHWC, 6, "split 1x4", 195, 303), (333, 26176, NHWC, 6, "split 1x4", 78, 145), (161, 48000, NHWC, 6, "split 2x2", 59, 67),
    (200, 41120, NHWC, 6, "split 1x4", 54, 60), (185, 16000, NCHW, 8, "wide", 24, 31), (145, 14720, NCHW, 4, "wide", 18, 23),
    (265, 12800, NCHW, 6, "wide", 33, 41), (510, 8192, NCHW, 4, "wide", 31, 53), (1001, 4096, NCHW, 8, "wide", 78, 136),
    (500, 17984, NCHW, 6, "split 1x4", 115, 150), (1000, 8992, NCHW, 6, "split 1x4", 198, 316), (129, 41600, NCHW, 6, "split 2x2", 45, 57),
])
def test_channel_counts_that_are_no_multiple_of_16(C, P, layout, bits, want, ahead, behind):
    assert form(C, P, layout, bits) == want, f"{ahead} us, {behind} in the other form"


@pytest.mark.parametrize("C,tiles,layout,bits,want,ahead,behind", [
    (512, 1456, NHWC, 6, "split 1x4", 23, 26), (512, 2304, NHWC, 6, "gemm8", 27, 33), (768, 1200, NHWC, 6, "gemm8", 33, 35),
    (1024, 1184, NHWC, 6, "gemm8", 42, 50), (1024, 1024, NHWC, 6, "split 1x4", 40, 42), (1024, 1024, NHWC, 8, "gemm8", 46, 51),
    (640, 1200, NHWC, 3, "split 1x4", 23, 28), (640, 900, NHWC, 8, "gemm8", 32, 37), (896, 784, NHWC, 8, "split 1x4", 38, 42),
    (144, 1535, NHWC, 8, "split 2x2", 12, 14), (192, 4092, NCHW, 6, "gemm4", 25, 29), (192, 2598, NCHW, 6, "split 2x2", 21, 22),
    (256, 4096, NCHW, 6, "gemm8", 24, 27), (256, 3800, NCHW, 6, "split 1x4", 23, 25), (400, 3497, NCHW, 6, "gemm4", 35, 37),
    (512, 3888, NCHW, 7, "split 1x4", 50, 64), (448, 3290, NCHW, 4, "split 1x4", 33, 40), (144, 4095, NCHW, 8, "gemm4", 27, 33), (640, 4080, NCHW, 6, "split 1x4", 70, 76),
])
def test_wide_tensors_of_whole_16_channels(C, tiles, layout, bits, want, ahead, behind):
    assert form(C, 32 * (tiles // -(-C // 32)), layout, bits) == want, f"{ahead} us, {behind} in the other form"


@pytest.mark.parametrize("C,P,bits,ahead,behind", [(128, 32992, 6, 14.5, 18.1), (128, 32992, 8, 18.3, 18.9), (128, 33600, 4, 13.4, 16.2),
                                                    (112, 32992, 6, 12.3, 15.5), (112, 33792, 6, 12.3, 15.4)])
def test_streaming_form_from_its_first_tile_on(C, P, bits, ahead, behind):
    """(A multiple of 16 channels; tensors with a few pixel tiles more than SIMDs were left to another form.)"""
    assert form(C, P, NHWC, bits).startswith("stream 4"), f"{ahead} us, {behind} in the other form"


def test_truncated_wide_tensors():
    assert form(768, 1344, NHWC, 8, 307) == "split 1x4"  # 25 us, 37 in the other form
    assert form(768, 1344, NHWC, 8, 700) == "gemm8"
    assert form(768, 4800, NCHW, 6, 40) == "split 1x4"
    assert form(512, 3200, NHWC, 6, 130) == "gemm8 fill"


@pytest.mark.parametrize("C,P,rows", [(97, 20800, 512), (64, 12288, 384), (250, 16384, 512), (161, 48000, 510), (353, 20000, 1023), (64, 3136, 196)])
def test_rows_of_counts_of_the_split_form(C, P, rows):
    """The table kernel adds them up in one workgroup: no more than run at once, where that costs the projection nothing."""
    assert fmtc.test_projection((1, 1, P, C), NHWC, 6).split(" nhwc ")[1] == str(rows)


def test_every_form_has_a_case():
    """The table of test_gpu_kernels holds every form that a tensor can take: a line that moves cannot leave a kernel untested."""
    pytest.importorskip("torch")
    from test_gpu_kernels import FORM_CASES, form_of

    reached = set()
    for C in range(1, 1025):
        ncs = -(-C // 32)
        for tiles in (50, 300, 1000, 1300, 1700, 2900, 3600, 4096, 4200, 17000):
            w = 32 * (tiles // ncs) // 21
            for layout in ("nhwc", "nchw"):
                for bits in (5, 8):
                    reached |= {form_of(fmtc, C, w, bits, layout, keep) for keep in (C, -(-C // 3))} if w else set()
    assert reached == {c[0] for c in FORM_CASES}
    for form, C, w, bits, *keep in FORM_CASES:
        assert form_of(fmtc, C, w, bits, form.rsplit(" ", 1)[1], *keep) == form


def test_arguments():
    for shape in ((0, 1, 1, 64), (1, 1, 1, 1025), (1 << 62, 4, 4, 64), (1 << 20, 8, 8, 64)):
        with pytest.raises(fmtc.FmtcError):
            fmtc.test_projection(shape, NHWC, 4)
    for bits, keep in ((1, 64), (9, 64), (4, 0), (4, 65)):
        with pytest.raises(fmtc.FmtcError):
            fmtc.test_projection((1, 1, 1, 64), NHWC, bits, keep)
