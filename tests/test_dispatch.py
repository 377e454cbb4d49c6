"""The lines of the dispatch rules: which kernel takes a call on either side of each (no GPU: see launches.py).  The
figures behind the lines stand beside the rules."""
import subprocess
import sys

import launches

LINEAR, CONV, DEPTHWISE = 0, 1, 2


def conv(B, hw, C, k, stride, Cout, pad=None):
    return (CONV, B, hw, hw, C, k, k, stride, k // 2 if pad is None else pad, Cout)


def check(cases):
    """cases: (operation, problem, start of the first kernel's name) each."""
    got = launches.calls([(op, p) for op, p, _ in cases])
    for (op, p, want), g in zip(cases, got):
        assert g[0].kernel.startswith(want), (op, p, g[0].kernel, "expected " + want)


def test_short_reductions_off_16_stay_with_the_tile_kernel():
    """The split-reduction kernel's 4-byte form: one round of the smallest tile that makes one, several while they take less time than
    the tile kernel's stages."""
    ks, tile = "hq_ksplit_kernel", "hq_gemm_kernel"
    small, rows, large = (ks + "<%s, false" % s for s in ("2, 2, 8, 1", "4, 2, 4, 1", "4, 4, 4, 1"))
    check([("fwd", conv(2, 28, 24, 1, 1, 96), small), ("fwd", conv(6, 28, 24, 1, 1, 96), rows), ("fwd", conv(20, 28, 100, 1, 1, 64), large),
           ("fwd", conv(26, 28, 56, 1, 1, 64), tile), ("fwd", conv(26, 28, 100, 1, 1, 64), tile),        # 20384 pixels, two rounds
           ("fwd", conv(26, 28, 200, 1, 1, 64), large),
           ("fwd", conv(13, 28, 56, 1, 1, 128), tile), ("fwd", conv(13, 28, 200, 1, 1, 128), large),
           ("fwd", conv(20, 10, 12, 3, 1, 256), rows), ("fwd", conv(16, 14, 36, 3, 1, 100), rows),
           ("fwd", conv(6, 28, 12, 3, 1, 256), tile), ("fwd", conv(6, 28, 100, 3, 1, 256), large),
           ("fwd", conv(26, 14, 12, 7, 1, 128), large), ("fwd", (LINEAR, 2058, 1, 1, 244, 1, 1, 1, 0, 760), large),
           ("fwd", conv(53, 28, 20, 3, 1, 16), rows), ("fwd", conv(61, 14, 760, 3, 1, 252), tile), ("fwd", conv(16, 14, 596, 3, 1, 160), rows),
           ("dgrad", (LINEAR, 16000, 1, 1, 128, 1, 1, 1, 0, 12), tile), ("dgrad", (LINEAR, 8000, 1, 1, 128, 1, 1, 1, 0, 12), large),
           ("dgrad", (LINEAR, 64, 1, 1, 128, 1, 1, 1, 0, 12), small)])


def test_strided_input_gradients_off_16_weigh_the_reduction_against_the_tiles():
    ks, tile = "hq_ksplit_kernel", "hq_gemm_kernel"
    check([("dgrad", conv(64, 112, 20, 1, 2, 20), tile), ("dgrad", conv(64, 112, 36, 1, 2, 36), tile),
           ("dgrad", conv(64, 112, 100, 1, 2, 100), tile), ("dgrad", conv(64, 112, 20, 3, 2, 20), ks),
           ("dgrad", conv(64, 112, 36, 3, 2, 36), ks), ("dgrad", conv(64, 112, 100, 3, 2, 100), ks),
           ("dgrad", conv(34, 25, 608, 1, 2, 24), tile), ("dgrad", conv(128, 56, 64, 1, 2, 200), ks),
           ("dgrad", conv(64, 28, 24, 1, 2, 24), ks), ("dgrad", conv(9, 50, 100, 3, 3, 12), tile),
           ("dgrad_sr", conv(64, 112, 36, 1, 2, 36), tile), ("dgrad", conv(8, 28, 100, 1, 2, 100), ks)])


def test_filters_of_more_than_64_taps_are_split():
    ks = "hq_ksplit_kernel"
    for layer in ((CONV, 4, 14, 14, 256, 9, 8, 1, 4, 64), (CONV, 4, 14, 14, 256, 8, 8, 1, 4, 64), (CONV, 2, 23, 21, 32, 11, 11, 2, 5, 48),
                  (CONV, 3, 13, 17, 20, 9, 8, 1, 4, 36), (CONV, 2, 19, 22, 12, 11, 11, 3, 5, 20)):
        check([(op, layer, ks) for op in ("fwd", "dgrad", "dgrad_sr", "dynamic_fwd")])
    # (offsets from a pixel's first tap that pass 2 GB are outside its arithmetic)
    check([("fwd", (CONV, 1, 3, 32768, 32768, 3, 1, 512, 0, 16), "hq_gemm_kernel<256, 32, 4, 1, 64, false, false"), ("fwd", (CONV, 1, 3, 21800, 32768, 3, 1, 512, 0, 16), ks)])
    # (taps times taps per row past 2^32 are outside the kernel's divisions)
    check([("fwd", (CONV, 1, 1, 70000, 16, 1, 65600, 1, 0, 16), "hq_gemm_kernel"), ("fwd", (CONV, 1, 1, 66000, 16, 1, 65500, 1, 0, 16), ks)])


def test_split_reductions_of_whole_chunks_end_where_the_tile_kernels_are_faster():
    def lin(M, k, n):
        return (LINEAR, M, 1, 1, k, 1, 1, 1, 0, n)
    ks, tile = "hq_ksplit_kernel", "hq_gemm_kernel"
    s32, small, large = (ks + "<%s, true" % s for s in ("2, 2, 8, 2", "2, 4, 8, 2", "4, 4, 8, 2"))
    check([("fwd", lin(2500, 512, 128), small), ("fwd", lin(2500, 256, 128), small), ("fwd", lin(5000, 512, 64), small),
           ("fwd", lin(5000, 240, 128), large), ("fwd", lin(5000, 256, 128), tile), ("fwd", lin(5000, 496, 128), tile), ("fwd", lin(5000, 512, 128), large),
           ("fwd", lin(12000, 256, 64), large), ("fwd", lin(8192, 1280, 128), large), ("fwd", lin(8193, 1040, 128), tile),
           ("fwd", conv(26, 28, 128, 3, 2, 128), large), ("fwd", conv(43, 28, 128, 3, 2, 128), "hq_ring_kernel"),
           ("fwd", conv(26, 14, 128, 3, 1, 128), large), ("fwd", conv(11, 14, 32, 7, 1, 200), large),
           ("fwd", conv(16, 28, 64, 5, 2, 200), large), ("fwd", conv(25, 28, 192, 5, 2, 200), tile),
           ("dgrad", conv(5, 28, 256, 1, 2, 256), large),                                          # strided: whatever the reduction
           # a second round under at most 64 channels and a long reduction
           ("fwd", lin(20000, 1024, 32), s32), ("fwd", lin(20000, 1008, 32), tile), ("fwd", lin(40000, 1024, 32), tile),
           ("fwd", lin(20000, 1024, 64), large), ("fwd", lin(33000, 1024, 64), tile), ("fwd", lin(16000, 1024, 80), tile),
           ("fwd", conv(60, 28, 128, 3, 2, 64), large), ("fwd", conv(102, 14, 128, 3, 1, 64), large)])
    # a strided input gradient's tiles are counted class by class: 242 pixels in four classes of 61, 61, 60 and 60
    # make 16 tiles of 16 pixels a column, not 16.0
    assert launches.calls([("dgrad", conv(2, 11, 504, 2, 2, 32, 0))])[0][0].blocks <= 256


def test_64_channel_layers_go_to_their_own_kernels_past_one_round():
    ks, regw, band, tile = "hq_ksplit_kernel", "hq_regw_kernel", "hq_band_kernel", "hq_gemm_kernel"
    check([(op, conv(20, 28, 64, 3, 1, 64), ks) for op in ("fwd", "dgrad", "dgrad_sr", "dynamic_fwd")] +
          [(op, conv(21, 28, 64, 3, 1, 64), regw) for op in ("fwd", "dgrad", "dgrad_sr", "dynamic_fwd")] +
          [("fwd", conv(10, 30, 64, 3, 1, 64, 0), ks), ("fwd", conv(21, 30, 64, 3, 1, 64, 0), band),                # no padding
           ("fwd", (CONV, 2, 20, 130, 64, 3, 3, 1, 1, 64), ks), ("fwd", (CONV, 7, 20, 130, 64, 3, 3, 1, 1, 64), regw),
           ("fwd", (CONV, 2, 30, 403, 64, 3, 3, 1, 1, 64), regw), ("fwd", (CONV, 2, 30, 404, 64, 3, 3, 1, 1, 64), tile),    # too wide for either
           ("fwd", conv(26, 28, 64, 3, 2, 64), ks), ("fwd", conv(90, 28, 64, 3, 2, 64), band), ("fwd", conv(20, 28, 64, 3, 2, 80), ks)])


def test_short_reductions_split_channels_for_want_of_pixels():
    point, tile = "hq_point_kernel", "hq_gemm_kernel"
    check([("fwd", (LINEAR, 40000, 1, 1, 192, 1, 1, 1, 0, 256), point), ("fwd", (LINEAR, 40000, 1, 1, 208, 1, 1, 1, 0, 256), tile),
           ("fwd", (LINEAR, 40000, 1, 1, 184, 1, 1, 1, 0, 256), tile), ("fwd", (LINEAR, 40000, 1, 1, 192, 1, 1, 1, 0, 248), tile),      # off 16
           ("fwd", (LINEAR, 40000, 1, 1, 128, 1, 1, 1, 0, 256), tile), ("dynamic_fwd", (LINEAR, 40000, 1, 1, 128, 1, 1, 1, 0, 256), point),
           # 128 channels: the general kernel's tiles are all resident, and more than a round and a third
           ("fwd", (LINEAR, 21760, 1, 1, 128, 1, 1, 1, 0, 256), point), ("fwd", (LINEAR, 21761, 1, 1, 128, 1, 1, 1, 0, 256), tile),
           ("fwd", (LINEAR, 65536, 1, 1, 128, 1, 1, 1, 0, 256), tile), ("fwd", (LINEAR, 65537, 1, 1, 128, 1, 1, 1, 0, 256), point),
           ("dgrad", (LINEAR, 40000, 1, 1, 256, 1, 1, 1, 0, 128), tile), ("dgrad_sr", (LINEAR, 40000, 1, 1, 256, 1, 1, 1, 0, 128), point),
           ("fwd", (LINEAR, 40000, 1, 1, 128, 1, 1, 1, 0, 240), point), ("fwd", (LINEAR, 40000, 1, 1, 96, 1, 1, 1, 0, 256), point),
           ("fwd", (LINEAR, 40000, 1, 1, 112, 1, 1, 1, 0, 256), point),
           ("fwd", conv(64, 57, 64, 1, 2, 64), point)])
    def blocks(*c):
        return launches.calls([("fwd", (LINEAR, c[0], 1, 1, c[1], 1, 1, 1, 0, c[2]))])[0][0].blocks
    assert blocks(401408, 32, 192) == 512 and blocks(8192, 192, 4096) == 512 and blocks(8192, 64, 512) == 256 and blocks(70000, 128, 512) == 512
    # stochastic rounding: channels split under any number of pixels
    layer = (LINEAR, 100244, 1, 1, 944, 1, 1, 1, 0, 64)
    assert [c[0].lds for c in launches.calls([("dgrad", layer), ("dgrad_sr", layer)])] == [30 * 2176, 6 * 2176]


def test_short_reductions_take_the_host_no_longer_for_more_channels():
    """The split is found among the numbers of 32-channel blocks that a workgroup's LDS holds, whatever the layer's number of channels."""
    code = """import sys, time, ctypes; rec = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL); sys.path.insert(0, sys.argv[2])
import paper_2105_04246_amd as hq
def least(n):
    p, best = hq.problem(hq.HQ_LINEAR, 2000, 1, 1, 16, 1, 1, 1, 0, n), 1.0
    for _ in range(50):
        rec.recorder_reset(0); t = time.perf_counter(); hq.hq_gemm_fwd(p, *[0x10000] * 9, 0); best = min(best, time.perf_counter() - t)
    return best
print(least(1 << 20) / least(1 << 10))"""
    r = subprocess.run([sys.executable, "-c", code, launches.recorder(), launches.ROOT], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stderr[-2000:]
    assert float(r.stdout) < 5, r.stdout                    # (50 when every split of the channels is tried)


def test_weight_gradients_of_few_blocks_are_streamed():
    import test_gpu_parity as T
    point, tile = "hq_wgrad_point_kernel", "hq_wgrad_kernel"
    lin = lambda m, c, n: (LINEAR, m, 1, 1, c, 1, 1, 1, 0, n)
    work = [(tuple(L)[1:], point) for L in T.POINT_WGRAD] + [(lin(16383, 32, 192), tile), (lin(40000, 32, 224), tile), (lin(65535, 224, 32), tile), (lin(99999, 32, 256), tile), (lin(200000, 32, 288), tile), (lin(40000, 96, 96), tile),
            (lin(40000, 48, 64), tile), (conv(60, 56, 64, 1, 2, 64), tile), (conv(128, 56, 32, 1, 1, 192), point)]
    for (p, want), got in zip(work, launches.calls([("wgrad", p) for p, _ in work])):
        assert [g.kernel.split("<")[0] for g in got] == ["zero_kernel", want, "wgrad_finalize_kernel"], (p, got)


def test_stochastic_rounding_takes_long_stages_while_all_tiles_are_resident():
    long_, short = "hq_gemm_kernel<128, 128, 2, 2, 128", "hq_gemm_kernel<128, 128, 2, 2, 64"
    check([("dgrad_sr", (LINEAR, 3255, 1, 1, 3624, 1, 1, 1, 0, 2064), short), ("dgrad", (LINEAR, 3255, 1, 1, 3624, 1, 1, 1, 0, 2064), long_),
           ("dgrad_sr", (LINEAR, 4096, 1, 1, 2048, 1, 1, 1, 0, 2064), long_), ("dgrad_sr", (LINEAR, 4096, 1, 1, 4096, 1, 1, 1, 0, 1040), short),
           ("dgrad_sr", conv(51, 28, 128, 1, 1, 288), short), ("dgrad_sr", conv(51, 28, 128, 1, 1, 256), long_),
           ("dgrad_sr", conv(60, 28, 96, 5, 2, 64), short), ("dgrad_sr", conv(41, 28, 256, 3, 2, 448), long_),
           ("dgrad_sr", conv(41, 28, 256, 3, 2, 256), short), ("dgrad_sr", conv(64, 28, 128, 5, 1, 64), short),
           ("dgrad_sr", conv(38, 28, 320, 1, 2, 1024), long_), ("dgrad_sr", (LINEAR, 5000, 1, 1, 1000, 1, 1, 1, 0, 300), short),
           ("dgrad_sr", (LINEAR, 3873, 1, 1, 1668, 1, 1, 1, 0, 3532), long_), ("dgrad_sr", (LINEAR, 5000, 1, 1, 2000, 1, 1, 1, 0, 1004), short),
           ("dgrad_sr", (LINEAR, 3187, 1, 1, 1544, 1, 1, 1, 0, 324), long_), ("dgrad_sr", (LINEAR, 3187, 1, 1, 1544, 1, 1, 1, 0, 316), short),
           ("dgrad_sr", (LINEAR, 900, 1, 1, 4000, 1, 1, 1, 0, 360), short), ("dgrad_sr", (LINEAR, 900, 1, 1, 4000, 1, 1, 1, 0, 436), long_)])


def test_whole_lines_per_stage_between_split_reductions_and_framed_tiles():
    ring, ks, tile, frame = "hq_ring_kernel", "hq_ksplit_kernel", "hq_gemm_kernel", "hq_frame_kernel"
    check([("fwd", conv(26, 14, 256, 3, 1, 256), frame), ("dgrad", conv(26, 14, 256, 3, 1, 256), frame), ("dgrad_sr", conv(26, 14, 256, 3, 1, 256), frame),
           ("dynamic_fwd", conv(26, 14, 256, 3, 1, 256), frame), ("fwd", conv(128, 4, 512, 3, 1, 512), ks),
           ("fwd", conv(257, 16, 128, 5, 1, 128), ring), ("fwd", conv(257, 32, 128, 3, 2, 128), ring),           # not the framed tiles' layers
           ("fwd", conv(257, 18, 128, 3, 1, 128, 0), ring), ("dgrad_sr", conv(257, 18, 128, 3, 1, 128, 0), ring),
           ("dgrad", conv(257, 32, 256, 3, 2, 256), tile),                                                      # strided
           ("fwd", (LINEAR, 8192, 1, 1, 1024, 1, 1, 1, 0, 1024), ring), ("fwd", (LINEAR, 8192, 1, 1, 896, 1, 1, 1, 0, 1024), tile),
           ("dgrad", (LINEAR, 8192, 1, 1, 1024, 1, 1, 1, 0, 1024), ring), ("dgrad_sr", (LINEAR, 8192, 1, 1, 1024, 1, 1, 1, 0, 1024), ring),
           ("dgrad", conv(42, 28, 128, 1, 1, 1024), ring),
           ("fwd", conv(26, 14, 192, 3, 1, 256), frame), ("fwd", conv(34, 13, 128, 3, 1, 144), frame), ("fwd", conv(128, 14, 256, 3, 1, 120), tile),
           ("fwd", conv(20, 30, 128, 3, 1, 144), frame), ("fwd", (LINEAR, 6700, 1, 1, 1024, 1, 1, 1, 0, 272), ring),
           ("fwd", (LINEAR, 1700, 1, 1, 1280, 1, 1, 1, 0, 1168), ring), ("fwd", conv(40, 29, 128, 3, 2, 272), ring),
           ("dgrad", conv(40, 16, 128, 3, 1, 128, 2), ring), ("fwd", (CONV, 20, 17, 19, 128, 5, 3, 1, 1, 160), ring),
           # the patch of a tile on wide images does not fit
           ("fwd", (CONV, 1, 70, 125, 128, 3, 3, 1, 1, 128), frame), ("fwd", (CONV, 1, 70, 126, 128, 3, 3, 1, 1, 128), ring),
           ("fwd", (CONV, 1, 70, 125, 192, 3, 3, 1, 1, 128), frame), ("fwd", (CONV, 1, 70, 126, 192, 3, 3, 1, 1, 128), tile),
           ("fwd", (CONV, 400, 1, 93, 192, 3, 3, 1, 1, 192), frame), ("dgrad_sr", (CONV, 400, 1, 94, 192, 3, 3, 1, 1, 192), tile)])


def test_framed_tiles_are_the_largest_that_fill_their_rounds():
    """Tiles of 128 to 512 pixels x 128 channels, one workgroup to a compute unit."""
    def tile(op, *layer):
        l = launches.calls([(op, conv(*layer))])[0][0]
        return l.kernel.split("<")[1][3:7], l.blocks
    assert tile("fwd", 128, 28, 128, 3, 1, 128) == ("4, 3", 224) and tile("fwd", 256, 28, 128, 3, 1, 128) == ("4, 3", 256)
    assert tile("dgrad", 256, 14, 256, 3, 1, 256) == ("4, 3", 224) and tile("dgrad_sr", 256, 7, 512, 3, 1, 512) == ("2, 2", 196)
    assert tile("fwd", 128, 32, 128, 3, 1, 128) == ("4, 4", 256) and tile("fwd", 128, 16, 256, 3, 1, 256) == ("2, 2", 256)
    assert tile("fwd", 128, 8, 512, 3, 1, 512) == ("1, 1", 256) and tile("fwd", 64, 14, 384, 3, 1, 384) == ("2, 1", 198)
    assert tile("dynamic_fwd", 60, 28, 128, 3, 1, 256) == ("3, 3", 246)


def test_whole_lines_of_one_tap_start_past_two_small_tiles_to_a_compute_unit():
    """64 x 64 tiles of the tile kernel: 512 or fewer keep it, with round-to-nearest-even below 10 lines."""
    ring, tile = "hq_ring_kernel", "hq_gemm_kernel"
    def lin(M, k, n, dgrad=True):
        return (LINEAR, M, 1, 1, n, 1, 1, 1, 0, k) if dgrad else (LINEAR, M, 1, 1, k, 1, 1, 1, 0, n)
    check([("dgrad", lin(8192, 1024, 256), tile), ("dgrad", lin(8193, 1024, 256), ring), ("dgrad", lin(8192, 1152, 256), tile), ("dgrad", lin(8192, 1280, 256), ring),
           ("fwd", lin(8192, 1152, 256, False), tile), ("fwd", lin(8192, 1280, 256, False), ring), ("fwd", lin(8193, 1024, 256, False), ring),
           ("dgrad_sr", lin(8192, 2048, 256), tile), ("dgrad_sr", lin(8193, 1024, 256), ring),
           ("dynamic_fwd", lin(8192, 2048, 256, False), tile), ("dynamic_fwd", lin(8193, 1024, 256, False), ring), ("dynamic_dgrad", lin(8193, 1024, 256), ring)])


def test_small_depthwise_launches_are_cut_into_short_strips():
    """Workgroups of the launch: a strip is a serial chain, so few threads get as many strips as there are rows."""
    def blocks(op, *layer):
        B, hw, C, stride = layer
        return max(l.blocks for l in launches.calls([(op, (DEPTHWISE, B, hw, hw, C, 3, 3, stride, 1, C))])[0] if l.kernel.startswith("hq_dw3x3"))
    for op, layer, want in (("dgrad_sr", (1, 14, 960, 2), 7 * 7), ("fwd", (2, 28, 32, 1), 28), ("dgrad", (1, 7, 32, 1), 7),
                            ("fwd", (8, 56, 192, 1), 42 * 14),      # at the line: strips of four rows
                            ("wgrad", (32, 7, 32, 1), 7), ("wgrad", (1, 7, 960, 2), 4), ("wgrad", (8, 28, 192, 1), 6 * 10), ("wgrad", (1, 112, 16, 1), 28)):
        assert blocks(op, *layer) == want, (op, layer, blocks(op, *layer))


def test_one_launch_weight_gradients_end_where_split_k_is_faster():
    one, split, band = "hq_wgrad_small_kernel", "zero_kernel", "hq_wgrad_band_kernel"
    check([("wgrad", conv(41, 28, 128, 3, 2, 64), split), ("wgrad", conv(33, 28, 128, 3, 2, 64), one),       # 8036, 6468 pixels: past and in the L2
           ("wgrad", conv(41, 28, 128, 3, 2, 128), one), ("wgrad", conv(41, 28, 256, 3, 2, 32), split),
           ("wgrad", conv(33, 28, 256, 3, 2, 32), one),
           ("wgrad", conv(41, 14, 16, 3, 1, 16), split), ("wgrad", conv(26, 14, 16, 3, 1, 16), one),
           ("wgrad", conv(41, 14, 64, 1, 1, 64), split), ("wgrad", conv(41, 14, 64, 1, 1, 128), one),
           ("wgrad", conv(41, 14, 64, 3, 1, 64), one), ("wgrad", conv(42, 14, 64, 3, 1, 64), band)])


def test_framed_weight_gradients_weigh_runs_against_slots():
    """Wide images as far as the ring fits LDS; one workgroup to a compute unit, and fewer where runs would be short."""
    band, tile = "hq_wgrad_band_kernel", "zero_kernel"
    check([("wgrad", (CONV, 1, 2, 570, 320, 3, 3, 1, 1, 256), band), ("wgrad", (CONV, 1, 2, 571, 320, 3, 3, 1, 1, 256), tile)])
    def blocks(*layer):
        return launches.calls([("wgrad", conv(*layer))])[0][0].blocks
    assert blocks(256, 56, 64, 3, 1, 64) == 2 * 128 and blocks(256, 7, 512, 3, 1, 512) == 128 * 2 and blocks(64, 14, 384, 3, 1, 384) == 72 * 3
    assert blocks(2000, 4, 64, 3, 1, 64) == 2 * 66                      # 391 units: runs of six


def test_tile_weight_gradients_load_without_branches_where_rows_are_whole_chunks():
    def kernel(*layer):
        return [l.kernel for l in launches.calls([("wgrad", layer)])[0] if l.kernel.startswith("hq_wgrad_kernel")][0]
    for layer, want in ((conv(46, 28, 80, 3, 2, 144), "<128, 128, false, false, true>"), (conv(13, 29, 48, 5, 1, 80), "<64, 64, false, false, true>"),
                        (conv(47, 14, 208, 1, 1, 96), "<128, 128, false, false, true>"), (conv(46, 28, 84, 3, 2, 144), "<128, 128, false, false, false>")):
        assert kernel(*layer).startswith("hq_wgrad_kernel" + want), (layer, kernel(*layer))


def test_first_layer_weight_gradients_stage_their_rows_under_every_stride():
    def kernels(*layer):
        return [l.kernel for l in launches.calls([("wgrad", layer)])[0]]
    for layer, want in (((CONV, 40, 33, 64, 3, 3, 3, 1, 1, 64), "hq_wgrad_stem_kernel<3>"), ((CONV, 9, 61, 64, 3, 7, 7, 3, 3, 64), "hq_wgrad_stem_kernel<3>"),
                        ((CONV, 4, 60, 60, 4, 4, 8, 1, 0, 64), "hq_wgrad_stem_kernel<4>"), ((CONV, 40, 33, 64, 3, 9, 3, 1, 1, 64), "hq_wgrad_kernel"),
                        ((CONV, 40, 33, 66, 3, 3, 3, 1, 1, 64), "hq_wgrad_kernel"), ((CONV, 40, 33, 64, 3, 3, 3, 1, 1, 80), "hq_wgrad_kernel")):
        assert any(k.startswith(want) for k in kernels(*layer)), (layer, kernels(*layer))


def test_small_first_layer_weight_gradients_are_cut_into_short_bands():
    def blocks(*layer):
        return [(l.kernel.split("<")[0], l.blocks) for l in launches.calls([("wgrad", layer)])[0] if not l.kernel.startswith(("zero", "wgrad_finalize"))]
    assert blocks(CONV, 1, 32, 32, 3, 7, 7, 1, 3, 32) == [("hq_wgrad_stem_kernel", 32)] and blocks(CONV, 4, 32, 32, 3, 7, 7, 1, 3, 32) == [("hq_wgrad_stem_kernel", 64)]
    assert blocks(CONV, 5, 28, 28, 3, 7, 7, 1, 3, 64) == [("hq_wgrad_stem_kernel", 50)]          # 140 rows: bands of three
    # large sums over few pixels, M = B * 11 * 23 under stride 1 and B * 7 * 13 under stride 2
    for B, c, n, stride, stem in ((2, 4, 64, 1, False), (23, 4, 64, 1, False), (24, 4, 64, 1, True), (2, 3, 64, 1, True), (2, 4, 48, 1, True),
                                  (65, 4, 64, 2, False), (66, 4, 64, 2, True)):
        assert (blocks(CONV, B, 12, 24, c, 8, 8, stride, 4 if stride == 2 else 3, n)[0][0] == "hq_wgrad_stem_kernel") == stem, (B, c, n, stride)


def test_column_sums_over_many_lines_are_shared():
    """hq_weight_prepare: a workgroup walks at most 8192 lines (rows of the weight tensor per tap) alone."""
    few, many = launches.calls([("weight_prepare", conv(1, 7, 512, 3, 1, 512)), ("weight_prepare", conv(1, 7, 64, 3, 1, 4096))])
    assert len(few) == 1 and len(many) == 2
    assert many[1].kernel == "weight_prepare_kernel" and many[1].blocks == 4 * 36
    one, words, stem = launches.calls([("weight_prepare", conv(1, 7, 4, 7, 1, 256)), ("weight_prepare", conv(1, 7, 36, 3, 1, 512)),
                                       ("weight_prepare", conv(1, 7, 3, 7, 2, 64))])
    assert (len(one), len(words), len(stem)) == (1, 2, 1)      # lines of 4 channels are read four at a time


def test_32_bit_pass_of_64_channel_layers():
    ks, regw = "hq_ksplit_kernel", "hq_regw_kernel"
    check([("dynamic_fwd", conv(7, 16, 64, 3, 1, 64), ks), ("dynamic_dgrad", conv(64, 16, 64, 3, 1, 64), ks),
           ("dynamic_fwd", conv(65, 16, 64, 3, 1, 64), regw), ("dynamic_fwd", conv(64, 16, 64, 3, 1, 128), regw),
           ("dynamic_fwd", conv(340, 7, 64, 3, 1, 64), regw)])


def test_32_bit_pass_of_first_layers_stores_whole_lines():
    got = launches.calls([("dynamic_fwd", conv(B, 56, 3, 3, 1, n)) for B, n in ((16, 16), (16, 32), (16, 48), (8, 48))] + [("fwd", conv(16, 56, 3, 3, 1, 48))])
    assert [g[0].kernel for g in got] == ["hq_stem_kernel<1, 0, 3, false>", "hq_stem_kernel<1, 2, 3, false>",
                                          "hq_stem_kernel<2, 2, 3, false>", "hq_stem_kernel<2, 0, 3, false>", "hq_stem_kernel<2, 1, 3, false>"]


def test_bands_of_first_layers_are_even_and_resident():
    """Workgroups of the launch: one per band up to 512."""
    def blocks(op, *c):
        return launches.calls([(op, conv(*c))])[0][0].blocks
    assert blocks("fwd", 130, 56, 3, 3, 1, 48) == 390 and blocks("fwd", 256, 56, 3, 3, 1, 48) == 512
    assert blocks("fwd", 100, 32, 3, 3, 1, 48) == 500              # not 800 bands of four rows in two uneven rounds
    assert blocks("fwd", 1, 224, 3, 7, 2, 64) == 112 and blocks("fwd", 300, 56, 3, 3, 1, 48) == 300
    assert blocks("dynamic_fwd", 100, 32, 3, 3, 1, 16) < 500


def test_every_gpu_of_a_process_is_told_of_large_lds():
    """The attribute that allows a kernel more dynamic LDS belongs to one GPU: a second GPU of the process needs it, too."""
    work = [("fwd", conv(128, 56, 64, 3, 1, 64)), ("dynamic_fwd", conv(128, 56, 64, 3, 1, 64)), ("dgrad_sr", conv(128, 56, 64, 3, 1, 64)),
            ("fwd", conv(128, 28, 128, 3, 1, 128)), ("dynamic_fwd", conv(128, 28, 128, 3, 1, 128)), ("dgrad_sr", conv(128, 28, 128, 3, 1, 128)),
            ("fwd", conv(128, 57, 64, 3, 2, 64)), ("fwd", conv(1, 7, 512, 3, 1, 512)), ("fwd", conv(26, 14, 128, 3, 1, 128)),
            ("fwd", (LINEAR, 256, 1, 1, 512, 1, 1, 1, 0, 512)), ("fwd", conv(64, 28, 256, 3, 2, 512)),
            ("wgrad", conv(128, 56, 64, 3, 1, 64)), ("wgrad", conv(64, 224, 3, 7, 2, 64)), ("wgrad", conv(64, 224, 4, 7, 2, 64)), ("wgrad", conv(3, 14, 256, 3, 1, 256)),
            ("wgrad", conv(20, 14, 256, 3, 1, 64))]
    got = launches.calls([(op, p, dev) for dev in (0, 1) for op, p in work])
    large = [l for calls in got[len(work):] for l in calls if l.lds > 48 * 1024]
    assert len({l.kernel for l in large}) >= 8
    for l in large:
        assert l.lds_allowed >= l.lds, l


def test_shapes_of_the_gpu_tests_reach_the_kernels_they_are_for():
    import test_gpu_parity as T
    def regw(op, s):
        B, H, W, C, n = s
        return launches.calls([(op, (CONV, B, H, W, C, 3, 3, 1, 1, n))])[0][0].kernel.startswith("hq_regw_kernel")
    assert all(regw(op, s) for s in T.REGW_ALL_MODES for op in ("dynamic_fwd", "dynamic_dgrad", "fwd", "dgrad", "dgrad_sr"))
    assert all(regw("fwd", s) for s in T.REGW_FORWARD)
    assert all(regw(op, s) for s in T.REGW_BACKWARD for op in ("dynamic_dgrad", "dgrad", "dgrad_sr"))
    assert all(regw("fwd", s) for s in T.REGW_RING_FORWARD)
    assert all(regw(op, s) for s in T.REGW_RING_BACKWARD for op in ("dynamic_dgrad", "dgrad", "dgrad_sr"))
    def point(op, s):
        B, H, W, C, stride, n = s
        return launches.calls([(op, (LINEAR if H * W == 1 else CONV, B, H, W, C, 1, 1, stride, 0, n))])[0][0].kernel.startswith("hq_point_kernel")
    assert all(point(op, s) for s in T.POINT_FORWARD for op in ("dynamic_fwd", "fwd"))
    assert all(point(op, s) for s in T.POINT_BACKWARD for op in ("dynamic_dgrad", "dgrad", "dgrad_sr"))
    assert not any(regw(op, s) for s in T.REGW_PAST + T.REGW_ONE_ROUND for op in ("dynamic_fwd", "fwd", "dgrad", "dgrad_sr"))
    for L in T.RING_BACKWARD + T.RING_OTHER:
        check([(op, tuple(L)[1:], "hq_frame_kernel" if L.R == 3 and L.pad == 1 else "hq_ring_kernel") for op in ("dgrad", "dgrad_sr", "dynamic_dgrad")])
    check([(op, tuple(L)[1:], "hq_frame_kernel") for L in T.FRAME_SHAPES for op in ("fwd", "dynamic_fwd")])
    check([(op, tuple(L)[1:], "hq_frame_kernel") for L in T.FRAME_SHAPES if L.Cout % 64 == 0 for op in ("dgrad", "dgrad_sr", "dynamic_dgrad")])
    assert {launches.calls([("fwd", tuple(L)[1:])])[0][0].kernel[16:23] for L in T.FRAME_SHAPES} == {"1, 1, 1", "1, 2, 1", "1, 2, 2", "1, 3, 3", "1, 4, 3", "1, 4, 4"}
    check([(op, tuple(L)[1:], "hq_gemm_kernel") for L in T.WIDE_IMAGES for op in ("fwd", "dgrad", "dgrad_sr", "dynamic_fwd")])
    check([("dgrad", tuple(L)[1:], "hq_ring_kernel") for L in T.RING_ONE_TAP])
    one, four = "hq_wgrad_small_kernel<1, 1, 4, 4>", "hq_wgrad_small_kernel<2, 2, 4, 2>"
    want = {"ws_1px": one, "ws_32_2145": one, "ws_32_300px": one, "ws_32_2304": one, "ws_64": four, "ws_64_256px": four, "past_ws_64": "zero_kernel",
            "past_ws_512": "zero_kernel", "ws_32x64": "hq_wgrad_small_kernel<1, 2, 8, 2>", "ws_8w": "hq_wgrad_small_kernel<1, 1, 8, 4>",
            "ws_16w_s2": "hq_wgrad_small_kernel<1, 1, 16, 2>"}
    lines = [L for L in T.WGRAD_LINES if L.name in want]
    assert len(lines) == len(want)
    for L, got in zip(lines, launches.calls([("wgrad", tuple(L)[1:]) for L in lines])):
        assert got[0].kernel == want[L.name], (L.name, got[0].kernel)


def test_names_in_the_benchmark_follow_the_dispatch():
    import bench
    import workloads as wl
    work = [(op, L) for net in (wl.resnet18_layers(B=256), wl.vgg16_layers(B=256)) for i, L in enumerate(net) for op in ("fwd", "dgrad", "wgrad") if i or op != "dgrad"]
    for (op, L), got in zip(work, launches.calls([(op, tuple(L)[1:]) for op, L in work])):
        names = [l.kernel.split("<")[0] for l in got if l.kernel != "zero_kernel"]
        assert bench.kernel_family(wl, L, op) == " + ".join(names), (op, L, names)
