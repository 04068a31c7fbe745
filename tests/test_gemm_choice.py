"""The rule that chooses a projection's kernel (twist_gemm_kernel, host only): never far from the fastest of the kernels as they were
measured on a MI355X."""
import ctypes
from dataclasses import replace

import pytest

import synth_inputs as si

NEVER = float("inf")  # more than three times the fastest: not measured
# layout, M, N, K, fp32 output, microseconds on tiles of 256x256, 256x128, 64x64 and 32x32 (operands in rotation, no cut)
UNCUT = [
    (1, 8192, 768, 64, 0, (8.0, 5.9, 12.1, 31.9)),
    (1, 8192, 768, 64, 1, (8.9, 8.0, 13.0, 33.2)),
    (1, 8192, 768, 128, 1, (10.3, 9.0, 13.5, 32.7)),
    (1, 8192, 768, 192, 1, (11.4, 10.0, 15.0, 35.6)),
    (1, 8192, 768, 256, 1, (12.3, 10.7, 15.7, 35.7)),
    (1, 8192, 768, 384, 1, (14.5, 12.5, 17.9, 39.8)),
    (0, 8192, 768, 64, 0, (8.4, 6.3, 11.6, 30.5)),
    (0, 8192, 768, 128, 1, (10.7, 9.4, 13.4, 31.4)),
    (0, 8192, 768, 192, 1, (11.9, 10.3, 14.2, 33.4)),
    (0, 8192, 768, 256, 1, (12.8, 11.1, 15.1, 33.3)),
    (0, 8192, 2048, 128, 0, (12.5, 13.5, 28.4, 75.7)),
    (0, 8192, 2048, 256, 0, (15.6, 17.4, 32.9, 81.8)),
    (0, 8192, 1024, 128, 0, (10.1, 8.1, 16.1, 40.1)),
    (1, 8192, 1024, 128, 0, (9.8, 7.8, 16.7, 42.3)),
    (1, 8192, 2048, 64, 0, (10.7, 11.0, 27.5, 81.0)),
    (1, 8192, 4096, 128, 0, (25.9, 25.4, 58.3, 162.8)),
    (1, 8192, 3072, 1024, 0, (56.9, 60.5, 108.6, 228.3)),
    (1, 8192, 3072, 2048, 1, (111.2, 121.7, 194.4, 393.2)),
    (1, 8192, 2048, 512, 1, (27.6, 33.6, 53.2, 112.0)),
    (1, 8192, 192, 768, 0, (22.1, 16.4, 9.2, 15.5)),
    (0, 4096, 768, 2560, 1, (57.1, 41.9, 29.9, 50.4)),
    (0, 4096, 768, 640, 1, (19.9, 14.7, 12.6, 23.3)),
    (0, 2048, 1536, 512, 1, (16.8, 12.8, 11.4, 22.1)),
    (0, 2048, 2048, 128, 0, (10.0, 7.6, 9.1, 21.7)),
    (0, 1000, 2048, 4096, 1, (78.7, 58.9, 28.7, 49.2)),
    (0, 1000, 512, 2048, 1, (43.5, 33.0, 10.3, 9.5)),
    (0, 512, 2048, 1024, 0, (24.9, 18.9, 7.4, 11.2)),
    (0, 128, 1536, 2048, 0, (42.6, 32.0, 9.9, 6.1)),
    (0, 33, 320, 1024, 1, (23.1, 17.5, 6.4, 4.2)),
    (0, 1, 768, 768, 0, (18.0, 13.7, 5.2, 3.9)),
    (0, 1, 192, 128, 1, (7.8, 5.9, 3.3, 3.1)),
    (1, 33, 768, 320, 0, (11.3, 7.9, 4.7, 3.7)),
    (1, 300, 1536, 64, 1, (8.2, 5.7, 4.0, 4.3)),
    (1, 1000, 1000, 4096, 0, (73.1, 58.0, 21.4, 39.1)),
    (1, 3000, 512, 768, 1, (20.7, 15.5, 9.7, 15.7)),
    (1, 4096, 512, 1024, 1, (23.5, 18.8, 11.7, 22.3)),
    (2, 64, 768, 4096, 1, (69.7, 59.8, 16.7, 12.5)),
    (2, 128, 512, 1000, 1, (24.5, 18.6, 6.6, 4.4)),
    (2, 1536, 1536, 2048, 1, (39.5, 33.8, 25.3, 47.5)),
    (2, 768, 4096, 1000, 1, (23.3, 19.7, 16.0, 33.2)),
    (2, 2048, 3072, 512, 1, (17.1, 15.2, 19.8, 45.7)),
    (2, 4096, 320, 512, 1, (17.3, 13.6, 7.7, 12.5)),
    (0, 8192, 50257, 64, 0, (340.4, 464.6, NEVER, NEVER)),
    (0, 3000, 50257, 64, 0, (128.5, 168.7, 205.1, NEVER)),
    (0, 8192, 32000, 64, 0, (127.5, 140.9, NEVER, NEVER)),
    (0, 1024, 50257, 64, 0, (56.2, 65.3, 81.7, NEVER)),
    (0, 1024, 50257, 768, 0, (126.3, 149.6, 191.6, NEVER)),
    (0, 7, 50257, 768, 0, (24.7, 30.8, 19.2, 20.7)),
    (0, 33, 32000, 256, 0, (12.6, 9.8, 7.1, 13.2)),
    (0, 3000, 1003, 64, 0, (20.3, 12.4, 8.4, 17.1)),
    (2, 50257, 64, 3000, 1, (87.2, 82.7, 88.9, 157.2)),
    (2, 32000, 256, 1024, 1, (28.0, 25.7, 49.0, NEVER)),
    (1, 1024, 256, 1024, 0, (NEVER, NEVER, 8.0, 5.3)),
    (0, 8192, 2304, 768, 0, (45.0, 46.0, 60.0, NEVER)),
]
# those of them, and of the products below, that run on tiles whose two groups of waves share the contraction: tile, microseconds there and on the fastest of the
# other kernels, cut where that pays, in one session
IN_GROUPS = {
    (0, 4096, 768, 2560, 1): ((128, 96), 24.2, 34.3),
    (0, 4096, 768, 640, 1): ((128, 96), 11.0, 12.7),
    (0, 2048, 1536, 512, 1): ((128, 96), 9.9, 11.1),
    (0, 1000, 2048, 4096, 1): ((128, 96), 26.5, 27.7),
    (2, 1536, 1536, 2048, 1): ((128, 128), 18.2, 22.9),
    (2, 768, 4096, 1000, 1): ((128, 128), 13.7, 15.2),
    (2, 2816, 2048, 8192, 1): ((192, 128), 93.7, 105.3),
    (2, 3072, 2048, 8192, 1): ((192, 128), 94.1, 106.2),
    (2, 2048, 768, 2048, 1): ((64, 96), 13.6, 15.4),
}
# TN products with scratch: those of (tile columns, parts of the contraction) within a quarter of the fastest, microseconds
CUT = [
    (768, 192, 8192, {(64, 6): 15.2, (64, 5): 15.2, (64, 4): 15.3, (64, 7): 15.4, (64, 3): 17.2, (64, 11): 17.9, (64, 14): 18.1, (64, 8): 18.2}),
    (768, 640, 4096, {(64, 2): 15.2, (64, 4): 16.7, (64, 3): 17.5, (64, 1): 17.5}),
    (256, 128, 2048, {(32, 1): 6.1, (32, 2): 7.6}),
    (512, 512, 4096, {(64, 4): 13.7, (64, 3): 13.8, (32, 1): 13.8, (64, 2): 15.5, (64, 8): 15.9, (64, 5): 16.1, (64, 7): 16.5, (64, 6): 16.9}),
    (512, 1024, 8192, {(64, 2): 22.3, (64, 6): 26.0, (64, 5): 26.5, (64, 3): 26.6, (64, 7): 26.9, (64, 4): 27.5}),
    (1024, 512, 1024, {(64, 1): 7.9, (32, 1): 8.3}),
    (2816, 2048, 8192, {(256, 2): 124.4}),
    (3072, 2048, 8192, {(256, 2): 126.6}),
    (2048, 896, 3000, {(64, 1): 22.8}),
    (2048, 768, 2048, {(64, 1): 16.8}),
    (3072, 768, 8192, {(256, 5): 62.3, (256, 6): 64.3, (256, 4): 65.7, (256, 7): 66.0, (128, 3): 73.2, (256, 3): 76.9}),
]


def _chosen(lib, cfg, *shape):
    h, out = ctypes.c_void_p(), (ctypes.c_int32 * 3)()
    d = lib.desc_from_cfg(cfg)
    assert lib.lib.twist_create(ctypes.byref(d), None, ctypes.byref(h)) == 0
    assert lib.lib.twist_gemm_kernel(h, *shape, out) == 0
    lib.lib.twist_destroy(h)
    return tuple(out)


# a fifth: two measurements of one product differ by up to a tenth, and so do the rule's estimates
@pytest.mark.parametrize("layout,M,N,K,f32,us", UNCUT)
def test_bf16_rule_is_near_the_fastest_kernel(lib, layout, M, N, K, f32, us):
    rows, cols, parts = _chosen(lib, si.CFG3, layout, M, N, K, f32, 0)
    if (layout, M, N, K, f32) in IN_GROUPS:
        tile, here, others = IN_GROUPS[layout, M, N, K, f32]
        assert (rows, cols, parts) == (*tile, 1) and here <= 1.2 * others
        return
    assert parts == 1 and us[((256, 256), (256, 128), (64, 64), (32, 32)).index((rows, cols))] <= 1.2 * min(us)


# products that tiles whose two groups of waves share the contraction make slower where their operands come from memory, and hardly faster otherwise: layout, M, N, K,
# fp32 output, tile, microseconds (operands in the caches, in memory) there and on those tiles
OTHERWISE = [
    (1, 1536, 1024, 4096, 0, (64, 64), (26.2, 29.9), (28.0, 36.4)),
    (1, 1504, 1088, 4480, 0, (64, 64), (29.2, 30.5), (30.2, 39.1)),
    (1, 3008, 576, 7744, 0, (64, 64), (49.2, 51.3), (48.6, 71.6)),
    (0, 1424, 576, 8128, 1, (64, 64), (30.2, 38.9), (33.1, 43.9)),
    (0, 8192, 2304, 768, 0, (256, 256), (43.5, 42.9), (40.1, 49.8)),
]


@pytest.mark.parametrize("layout,M,N,K,f32,tile,here,others", OTHERWISE)
def test_bf16_rule_minds_operands_in_memory(lib, layout, M, N, K, f32, tile, here, others):
    assert sum(here) < sum(others) and _chosen(lib, si.CFG3, layout, M, N, K, f32, 0) == (*tile, 1)


@pytest.mark.parametrize("M,N,K,us", CUT)
def test_bf16_rule_cuts_a_contraction_where_it_pays(lib, M, N, K, us):
    rows, cols, parts = _chosen(lib, si.CFG3, 2, M, N, K, 1, 1 << 24)
    if (2, M, N, K, 1) in IN_GROUPS:
        tile, here, others = IN_GROUPS[2, M, N, K, 1]
        assert (rows, cols, parts) == (*tile, 1) and here <= 1.2 * others
        return
    assert (cols, parts) in us, (cols, parts)


def test_a_product_is_cut_only_into_the_scratch_it_has(lib):
    for cfg in (si.CFG1, si.CFG3):
        assert _chosen(lib, cfg, 2, 768, 192, 8192, 1, 0)[2] == 1
        parts = _chosen(lib, cfg, 2, 768, 192, 8192, 1, 1 << 24)[2]
        assert parts > 1 and _chosen(lib, cfg, 2, 768, 192, 8192, 1, parts * 768 * 192 - 1)[2] < parts
    assert _chosen(lib, si.CFG3, 0, 768, 192, 8192, 1, 1 << 24)[2] == 1


def test_fp32_rule_leaves_short_contractions_of_large_outputs_to_the_plain_kernel(lib):
    assert _chosen(lib, si.CFG1, 0, 8192, 2048, 8, 1, 0)[0] == 0 and _chosen(lib, si.CFG1, 0, 512, 50257, 16, 1, 0)[0] == 0
    assert _chosen(lib, si.CFG1, 2, 3072, 768, 8, 1, 0)[0] == 0 and _chosen(lib, si.CFG1, 2, 4096, 4096, 16, 1, 0)[0] == 128
    assert _chosen(lib, si.CFG1, 0, 8192, 2048, 17, 1, 0)[0] == 128 and _chosen(lib, si.CFG1, 2, 768, 768, 8, 1, 0)[0] == 32


# cfg, tokens, columns of heads and of the FFN's hidden layer -> microseconds of a pass of 6 layers (3 from 600 GFLOP a layer) as measured on a MI355X, weight
# gradients in one launch a layer, on the second stream apart, the FFN's paired, the attention's paired, both paired
FORMS = [
    (si.CFG3, 2048, 8192, 1024, 2816, (10142, 9853, 10417, 9818, 10396)),
    (si.CFG2, 768, 2048, 512, 2048, (1472, 1596, 1543, 1574, 1543)),
    (si.CFG2, 768, 8192, 192, 768, (2101, 2295, 2252, 2243, 2216)),
    (si.CFG2, 768, 2048, 384, 1536, (1317, 1475, 1401, 1458, 1390)),
    (si.CFG2, 768, 2048, 768, 704, (1347, 1484, 1470, 1436, 1440)),
    (si.CFG2, 768, 8192, 768, 3072, (4938, 5301, 5207, 5208, 5110)),
    (si.CFG3, 768, 2048, 384, 1056, (1275, 1436, 1363, 1423, 1353)),
    (si.CFG3, 1024, 1024, 1024, 1408, (1450, 1569, 1538, 1594, 1587)),
    (si.CFG2, 1600, 8192, 768, 3200, (7529, 7334, 7164, 7219, 7135)),
    (si.CFG2, 1536, 2048, 384, 3072, (2349, 2444, 2340, 2364, 2270)),
    (si.CFG2, 1536, 3000, 1536, 3072, (4150, 4029, 3989, 3860, 3830)),
    (si.CFG3, 1536, 3000, 1536, 2112, (4176, 3969, 3872, 3829, 3795)),
    (si.CFG3, 2048, 1024, 512, 5632, (3274, 3095, 3182, 3117, 3215)),
    (si.CFG3, 2048, 4096, 1408, 2816, (6732, 6506, 6773, 6515, 6822)),
    (si.CFG3, 3072, 2048, 2048, 4224, (6580, 6326, 6377, 6267, 6309)),
    (si.CFG2, 3072, 3000, 1536, 3072, (6666, 5992, 6261, 6026, 6307)),
    (si.CFG3, 4096, 8192, 2688, 5632, (17226, 16448, 16762, 16655, 16896)),
]


# 3 %: two runs of one form differ by up to 2
@pytest.mark.parametrize("cfg,d,tokens,heads,ffn,us", FORMS)
def test_weight_gradients_take_nearly_the_fastest_form(lib, cfg, d, tokens, heads, ffn, us):
    h, out = ctypes.c_void_p(), (ctypes.c_int32 * 4)()
    desc = lib.desc_from_cfg(replace(cfg, d_model=d))
    assert lib.lib.twist_create(ctypes.byref(desc), None, ctypes.byref(h)) == 0
    assert lib.lib.twist_backward_schedule(h, tokens, heads, ffn, out) == 0
    lib.lib.twist_destroy(h)
    assert us[0 if out[0] else 1 + out[1] + 2 * out[2]] <= 1.03 * min(us)


# cfg, tokens, columns of heads and of the FFN's hidden layer in an average layer -> (one launch on the caller's stream, FFN paired, attention paired)
@pytest.mark.parametrize("cfg,tokens,heads,ffn,want", [
    (si.CFG3, 8192, 1024, 2816, (0, 0, 1)), (si.CFG3, 3000, 896, 2488, (0, 1, 1)), (si.CFG2, 2048, 384, 1536, (1, 1, 1)), (si.CFG2, 2048, 768, 704, (1, 1, 1)),
    (si.CFG2, 8192, 192, 768, (1, 1, 1)), (replace(si.CFG3, d_model=1024), 2048, 512, 1408, (1, 1, 1)), (replace(si.CFG3, d_model=1024), 256, 512, 1408, (1, 0, 0)),
    (replace(si.CFG2, dtype="f32"), 1024, 384, 1536, (0, 0, 0)), (si.CFG1, 256, 64, 256, (1, 0, 0))])
def test_schedule_of_the_weight_gradients(lib, cfg, tokens, heads, ffn, want):
    h, out = ctypes.c_void_p(), (ctypes.c_int32 * 4)()
    d = lib.desc_from_cfg(cfg)
    assert lib.lib.twist_create(ctypes.byref(d), None, ctypes.byref(h)) == 0
    assert lib.lib.twist_backward_schedule(h, tokens, heads, ffn, out) == 0
    assert tuple(out)[:3] == want and out[3] == (not want[0])
    assert lib.lib.twist_set_overlap(h, 0) == 0 and lib.lib.twist_backward_schedule(h, tokens, heads, ffn, out) == 0 and out[3] == 0
    assert lib.lib.twist_backward_schedule(h, 0, heads, ffn, out) == 1
    lib.lib.twist_destroy(h)
