"""What the dispatchers of the dense layers and of attention decide, asked of the library without a GPU (it then plans for 256 compute units)."""
import ctypes as C

import pytest

from paper_2110_14895_amd import binding

EPI_BIAS, EPI_BIAS_GELU, EPI_BIAS_RESID, EPI_PARTIAL = 0, 1, 2, 4       # EpEpilogue


class DensePlan(C.Structure):
    _fields_ = [("splits", C.c_int32), ("persistent", C.c_int32), ("bm", C.c_int32), ("bn", C.c_int32), ("per_cu", C.c_int32),
                ("m_main", C.c_int64)]

    def __str__(self):
        """rows x columns of a tile; x2: two workgroups to a unit; P: the persistent kernel, + rows past its walk; / K ranges"""
        return ("P" if self.persistent else "") + f"{self.bm}x{self.bn}" + ("x2" if self.per_cu == 2 else "") + \
            (f"/{self.splits}" if self.splits > 1 else "")


def dense_plan(rows, n, k, epi, one_order=False):
    p = DensePlan()
    f = binding.lib().ep_query_dense_plan_one_order if one_order else binding.lib().ep_query_dense_plan
    f.argtypes, f.restype = [C.c_int64, C.c_int32, C.c_int32, C.c_int32, C.POINTER(DensePlan)], None
    f(rows, n, k, epi, C.byref(p))
    return p


# widths of the named shapes, then wide MLPs and narrow models with a long K
@pytest.mark.parametrize("d,m,t", [(384, 1536, 197), (768, 3072, 197), (1024, 4096, 197), (1280, 5120, 257),
                                   (1024, 16384, 197), (2048, 16384, 257), (2048, 32640, 50), (64, 8192, 257), (448, 7168, 197)])
def test_sums_over_k_ranges_stay_bounded(d, m, t):
    cut = 0
    for b in range(1, (1 << 17) // t):
        p = dense_plan(b * t, d, m, EPI_PARTIAL)
        cut += p.splits > 1
        if p.splits > 1:
            assert p.splits * b * t * d * 4 <= 32 << 20 and b * t <= 1 << 15, (b, p.splits)
            assert m % (64 * p.splits) == 0 and m // 64 // p.splits >= 8
    assert cut > 0


# A few hundred rows past the tile walk cost more than the round of tiles they save: q|k|v and first MLP layer of several
# widths, once as slow as 1.5 times the launch that covers all rows
@pytest.mark.parametrize("rows,n,k,epi", [(3859, 4608, 1536, EPI_BIAS), (3380, 16384, 2048, EPI_BIAS_GELU), (4039, 5760, 1920, EPI_BIAS),
                                          (9135, 3840, 1280, EPI_BIAS_GELU), (7410, 2304, 768, EPI_BIAS)])
def test_no_long_tails_of_narrow_tiles(rows, n, k, epi):
    p = dense_plan(rows, n, k, epi)
    assert rows - p.m_main <= 64


# one round of 256-row tiles and more, fp32 output with a residual: 5 to 17 % faster on the persistent kernel than as
# 256 x 256 tiles of a workgroup each
@pytest.mark.parametrize("rows,n,k", [(12850, 1280, 1280), (23443, 1280, 1280), (57825, 1280, 5120), (20560, 768, 768), (33884, 2048, 2048)])
def test_large_residual_layers_run_on_the_persistent_kernel(rows, n, k):
    assert dense_plan(rows, n, k, EPI_BIAS_RESID).persistent


# A tile's rows of the output are addressed with 32 bits up to 2^20 columns; wider layers (embeddings) run as 64 x 32 tiles
@pytest.mark.parametrize("n", [(1 << 20) - 64, 1 << 20, 1052736, 1500032, 1 << 21, (1 << 22) + 64])
def test_layers_of_a_million_columns_do_not_run_on_the_persistent_kernel(n):
    for k in (64, 128, 192, 960):
        for rows in (1, 64, 255, 256, 300, 511, 512, 1000, 2047):
            if rows * n >= 1 << 31 or n * k * 2 >= 0x7FFFFFF0:
                continue
            for epi in (EPI_BIAS, EPI_BIAS_GELU, EPI_BIAS_RESID):
                assert n < 1 << 20 or not dense_plan(rows, n, k, epi).persistent, (rows, k, epi)


def group_limit(d, heads, m, t, micro, in_dtype=binding.EP_F32, param_dtype=binding.EP_BF16):
    cfg = binding.VitConfig(1, d, heads, m, t, 1e-6, param_dtype, in_dtype, binding.EP_F32).c_struct()
    f = binding.lib().ep_query_group_limit
    f.argtypes, f.restype = [C.c_void_p, C.c_int32], C.c_int32
    return f(C.addressof(cfg), micro)


# Micro-batches that a pipeline takes together get the bits of each on its own: neither alone nor together may a dense layer
# have narrow tiles, whose sums are put together otherwise (a second MLP layer cut into K ranges never has)
@pytest.mark.parametrize("in_dtype", [binding.EP_F32, binding.EP_BF16])
@pytest.mark.parametrize("d,heads,m,t", [(192, 3, 768, 197), (384, 6, 1536, 197), (512, 8, 2048, 197), (768, 12, 3072, 197),
                                         (768, 12, 3072, 577), (1024, 16, 4096, 197), (1280, 16, 5120, 257)])
def test_grouped_micro_batches_have_no_narrow_tiles(d, heads, m, t, in_dtype):
    grouped = alone = 0
    for micro in range(1, 16384 // t + 2):
        rows, limit = micro * t, group_limit(d, heads, m, t, micro, in_dtype)
        layers = [(d, d, EPI_BIAS_RESID)]
        if d > 384 or in_dtype == binding.EP_BF16:           # otherwise LayerNorm goes with them
            layers.append((3 * d, d, EPI_BIAS))
        if d > 384:
            layers.append((m, d, EPI_BIAS_GELU))
        if dense_plan(rows, d, m, EPI_PARTIAL).splits == 1:
            layers.append((d, m, EPI_BIAS_RESID))
        if limit == 1:
            alone += any(dense_plan(rows, *l).m_main < rows for l in layers)
            continue
        assert rows <= 1 << 14
        grouped += 1
        for n in range(1, limit + 1):
            for l in layers:
                assert dense_plan(n * rows, *l, one_order=n > 1).m_main == n * rows, (micro, n, l)
    assert grouped > 0
    assert alone > 0 or d <= 384


def test_what_is_not_grouped():
    assert group_limit(192, 3, 768, 197, 8, param_dtype=binding.EP_F32) == 1            # fp32
    assert group_limit(384, 6, 1536, 577, 28) == 2 and group_limit(384, 6, 1536, 577, 29) == 1         # 2^14 rows
    assert group_limit(768, 12, 3072, 197, 41) > 1 and group_limit(768, 12, 3072, 197, 42) == 1        # narrow tiles alone


def f32_ln_route(rows, n, k, cus=256):
    f = binding.lib().ep_query_f32_ln_route
    f.argtypes, f.restype = [C.c_int64, C.c_int32, C.c_int32, C.c_int32], C.c_int32
    return f(rows, n, k, cus)


# fp32 LayerNorm and dense layer: 0 in two launches (the rows kernel up to 1.6 times as long), 3 rows in registers (two launches
# up to 1.6 times as long), 1 and 2 tiles of 16 and 32 that normalise on the way
@pytest.mark.parametrize("rows,n,k,route", [
    (65, 768, 192, 1), (591, 768, 192, 2), (394, 288, 96, 1),
    (25216, 768, 96, 0), (9456, 1600, 200, 0), (6304, 1792, 224, 0), (25216, 1600, 160, 0), (12608, 1536, 384, 0), (2364, 2560, 320, 0),
    (12608, 96, 32, 3), (25216, 256, 32, 3), (6304, 768, 192, 3), (25216, 192, 64, 3), (394, 1536, 384, 3), (1182, 600, 200, 3),
])
def test_fp32_layernorm_and_dense_layer(rows, n, k, route):
    assert f32_ln_route(rows, n, k) == route


@pytest.mark.parametrize("pairs", [1, 2, 16, 24, 32, 36, 60, 96, 128, 140, 255, 256, 257, 272, 4096])
def test_every_attention_group_holds_a_query(pairs):
    f = binding.lib().ep_query_attention_plan
    f.argtypes, f.restype = [C.c_int64, C.c_int32, C.c_int32, C.POINTER(C.c_int32), C.POINTER(C.c_int32)], None
    qw, ng = C.c_int32(), C.c_int32()
    for t in list(range(1, 1200)) + [2049, 4096]:
        f(pairs, t, 256, C.byref(qw), C.byref(ng))
        tiles = -(-t // qw.value)
        to_a_group = -(-tiles // ng.value)
        assert qw.value in (16, 32) and 1 <= to_a_group <= 10, t        # the query waves of a workgroup
        assert (ng.value - 1) * to_a_group < tiles, t
        assert pairs * ng.value <= 256 or ng.value == -(-t // 320), t   # one round of units, or as few groups as fit


def ln_plan(rows, n, k, epi):
    """Rows of a panel and column groups of LayerNorm and a dense layer in one launch; (0, 0): two launches."""
    f = binding.lib().ep_query_ln_gemm_plan
    f.argtypes, f.restype = [C.c_int64, C.c_int32, C.c_int32, C.c_int32, C.c_int32, C.POINTER(C.c_int32)], C.c_int32
    groups = C.c_int32()
    return f(rows, n, k, epi, 256, C.byref(groups)), groups.value


# In one launch with its LayerNorm a wide MLP's first layer takes up to 1.5 times as long, and so do some of few rows or little more than a round
@pytest.mark.parametrize("rows,n,k,one", [
    (394, 1152, 384, 0), (500, 6144, 384, 1), (600, 12288, 384, 0), (1024, 12288, 384, 1), (17, 8192, 256, 1),
    (499, 1536, 512, 0), (500, 4096, 512, 1), (606, 6144, 512, 0), (1000, 8192, 512, 1), (8080, 16384, 512, 0), (20001, 2048, 512, 0),
    (1899, 3072, 768, 0), (1900, 3072, 768, 1), (1899, 9216, 768, 0), (1900, 9216, 768, 1), (2599, 3056, 768, 0), (2600, 3056, 768, 1), (2000, 9232, 768, 0),
    (2599, 2304, 768, 0), (2600, 9216, 768, 1), (9595, 12288, 768, 0), (10240, 3072, 768, 1), (10241, 3072, 768, 0), (10302, 2304, 768, 1),
    (10752, 3072, 768, 0), (10753, 6144, 768, 1), (11110, 9216, 768, 0), (20001, 2304, 768, 0),
    (1750, 4096, 1024, 0), (3152, 4096, 1024, 0), (4616, 4096, 1024, 0), (4950, 4096, 1024, 0),       # up to 1.05 where weights are not touched
    (5499, 1024, 1024, 0), (5500, 2304, 1024, 1), (5888, 4096, 1024, 0), (5889, 4096, 1024, 1), (6363, 5120, 1024, 0), (8192, 16384, 1024, 0),
    (8193, 3072, 1024, 0), (5632, 3072, 1024, 1), (5633, 3072, 1024, 0), (6400, 3072, 1024, 0), (6401, 3072, 1024, 1), (5888, 2816, 1024, 0),
    (5889, 2816, 1024, 1), (1576, 2304, 576, 0), (6304, 2688, 896, 0),
])
def test_layernorm_and_dense_layer_in_one_launch(rows, n, k, one):
    assert all((ln_plan(rows, n, k, epi)[0] > 0) == one for epi in (EPI_BIAS, EPI_BIAS_GELU))


# Panels of 32 rows: first MLP layers (with GELU) of narrow models on few rows and no other layer
@pytest.mark.parametrize("rows,n,k,few", [
    (2560, 768, 192, 1), (2561, 768, 192, 0), (1, 256, 64, 1), (1, 240, 64, 0), (2473, 1536, 384, 1), (2474, 1536, 384, 0),     # 2560 rows, 4 K, 3.8 million outputs
    (197, 6144, 384, 1), (197, 6160, 384, 0), (17, 5120, 320, 1), (17, 5136, 320, 0), (17, 16384, 256, 1),                      # 16 K past 256 wide
    (197, 2048, 512, 0), (257, 14784, 256, 1), (257, 14800, 256, 0),
])
def test_panels_of_few_rows(rows, n, k, few):
    assert (ln_plan(rows, n, k, EPI_BIAS_GELU)[0] == 32) == few
    assert ln_plan(rows, n, k, EPI_BIAS)[0] != 32


# A first MLP layer at 1024 wide whose weights attention has touched: in one launch with its LayerNorm where its own would be one round of
# 256 x 256 tiles on 193 to 208 of 256 units; nothing else moves
@pytest.mark.parametrize("rows,n,one", [
    (3072, 4096, 0), (3073, 4096, 1), (3152, 4096, 1), (3328, 4096, 1), (3329, 4096, 0), (2880, 4352, 0), (2881, 4160, 1), (3072, 4352, 1), (3073, 4352, 0),
    (2955, 4416, 0), (3840, 3136, 0), (3841, 3136, 1), (4096, 3136, 1), (4097, 3136, 0), (4000, 3072, 0), (3264, 3840, 0), (3265, 3840, 1), (3152, 3840, 0),
    (4616, 4096, 0), (5888, 4096, 0), (5889, 4096, 1),
])
def test_layernorm_and_touched_first_mlp_layer(rows, n, one):
    f = binding.lib().ep_query_ln_gemm_touched_mlp
    f.argtypes, f.restype = [C.c_int64, C.c_int32, C.c_int32], C.c_int32
    assert f(rows, n, 1024) == one
    if rows < 5500:
        assert ln_plan(rows, n, 1024, EPI_BIAS_GELU)[0] == 0
        p = dense_plan(rows, n, 1024, EPI_BIAS_GELU)
        assert not one or (p.m_main == rows and str(p) == "256x256")             # no rows that add up in another order
    for k in (320, 512, 768):
        assert f(rows, n, k) == (ln_plan(rows, n, k, EPI_BIAS_GELU)[0] > 0)


# Narrow models of many rows: several column groups in two rounds where one round of 128-row panels leaves units without work
@pytest.mark.parametrize("rows,n,k,epi,plan", [
    (16383, 1536, 384, EPI_BIAS_GELU, (64, 1)), (20037, 1536, 384, EPI_BIAS_GELU, (128, 3)), (21814, 2048, 256, EPI_BIAS_GELU, (64, 2)),
    (23279, 960, 320, EPI_BIAS, (64, 2)),
    (22458, 1536, 384, EPI_BIAS_GELU, (128, 1)), (34249, 1536, 384, EPI_BIAS_GELU, (64, 1)), (34249, 3072, 384, EPI_BIAS_GELU, (64, 2)),
    (22458, 1536, 192, EPI_BIAS_GELU, (64, 2)), (36053, 1536, 192, EPI_BIAS_GELU, (64, 2)), (50432, 1152, 384, EPI_BIAS, (128, 1)), (50432, 768, 192, EPI_BIAS_GELU, (128, 1)),
])
def test_panels_of_many_narrow_rows(rows, n, k, epi, plan):
    assert ln_plan(rows, n, k, epi) == plan


# Heights between the table's past the layers that they were fitted to: long K keeps one round of wide tiles, few rows without GELU keep theirs
@pytest.mark.parametrize("rows,n,k,epi,shape", [
    (12462, 1024, 12800, EPI_BIAS_RESID, "256x256"), (8312, 1536, 30784, EPI_BIAS_RESID, "256x256"), (5504, 2048, 21568, EPI_BIAS_RESID, "256x192"),
    (11212, 1024, 25792, EPI_BIAS_RESID, "192x256"), (157, 12288, 3072, EPI_BIAS, "128x128"), (146, 1536, 28160, EPI_PARTIAL, "128x128/8"),
    (199, 12288, 768, EPI_BIAS, "128x128"),
    # on either side of the lines, and long K in more than a round or on narrow tiles
    (6400, 1536, 5120, EPI_BIAS_RESID, "256x192"), (5757, 1536, 6144, EPI_BIAS_RESID, "144x128"), (19823, 1024, 28992, EPI_BIAS_RESID, "208x128"), (2188, 1280, 12736, EPI_BIAS_RESID, "96x128"),
    (259, 1280, 25600, EPI_PARTIAL, "96x128/8"), (184, 15360, 1280, EPI_BIAS_GELU, "96x128"),
])
def test_heights_past_their_fit(rows, n, k, epi, shape):
    assert str(dense_plan(rows, n, k, epi)) == shape


# One round of wide tiles whose outputs fill three quarters of the chip is the faster one inside a stage, and so is any at 768 columns
@pytest.mark.parametrize("rows,n,k,shape", [
    (10280, 1280, 5120, "256x256"), (12608, 1024, 4096, "256x256"), (9456, 1024, 4096, "256x192"), (9850, 1024, 4096, "256x192"), (11032, 768, 3072, "256x192"),
    (9595, 1024, 8192, "256x192"), (7575, 1280, 5120, "256x192"),
    (8989, 1024, 4096, "144x128"), (6868, 1280, 5120, "144x128"), (5555, 1536, 6144, "144x128"), (19700, 1024, 4096, "208x128"),
])
def test_one_round_of_wide_residual_tiles(rows, n, k, shape):
    assert str(dense_plan(rows, n, k, EPI_BIAS_RESID)) == shape


class TouchPlan(C.Structure):
    _fields_ = [("kind", C.c_int32), ("begin", C.c_int64), ("end", C.c_int64), ("layer_bytes", C.c_int64), ("weights", C.c_int64 * 4),
                ("weight_ends", C.c_int64 * 4)]


TOUCH_NONE, TOUCH_LONG, TOUCH_ALL = 0, 1, 2


def touch_plan(d, heads, m, t, batch, ranges_of=0, next_layer=True, param_dtype=binding.EP_BF16):
    """Which weights attention touches for the launches behind it, and where they lie from where the layer begins."""
    cfg = binding.VitConfig(1, d, heads, m, t, 1e-6, param_dtype, param_dtype, binding.EP_F32).c_struct()
    f, p = binding.lib().ep_query_touch_plan, TouchPlan()
    f.argtypes, f.restype = [C.c_void_p, C.c_int32, C.c_int32, C.c_int32, C.POINTER(TouchPlan)], None
    f(C.addressof(cfg), batch, ranges_of, next_layer, C.byref(p))
    return p


# either side of every line of the rule
@pytest.mark.parametrize("d,heads,m,t,batch,kind", [
    (768, 12, 3072, 382, 1, TOUCH_NONE), (768, 12, 3072, 383, 1, TOUCH_ALL),                # 27 rows to a MB of weights
    (1024, 16, 4096, 283, 4, TOUCH_NONE), (1024, 16, 4096, 103, 11, TOUCH_LONG),            # 45 where the second MLP layer is cut into ranges
    (1280, 16, 5120, 61, 29, TOUCH_NONE), (1280, 16, 5120, 59, 30, TOUCH_LONG), (1280, 16, 5120, 8, 200, TOUCH_LONG),       # uncut: 27 again
    (1024, 16, 4096, 173, 16, TOUCH_LONG), (1024, 16, 4096, 213, 13, TOUCH_ALL),            # 110
    (768, 12, 3072, 50, 16, TOUCH_ALL), (832, 13, 3328, 50, 16, TOUCH_LONG),                # up to 768 wide all of them
    (768, 12, 42112, 100, 41, TOUCH_ALL), (768, 12, 42176, 100, 41, TOUCH_NONE),            # 128 MB
    (1152, 18, 4608, 1000, 8, TOUCH_ALL), (1216, 19, 4864, 1000, 8, TOUCH_NONE),            # 256 x 192 tiles: 32 MB
    (1024, 16, 4096, 8, 512, TOUCH_ALL), (1024, 16, 4096, 8, 513, TOUCH_NONE),              # a persistent first MLP layer
    (1024, 16, 4096, 8, 1750, TOUCH_NONE),                                                  # a persistent second one
    (128, 2, 256, 288, 140, TOUCH_ALL), (128, 2, 256, 320, 140, TOUCH_NONE), (1024, 16, 4096, 577, 6, TOUCH_NONE),          # ten query waves
])
def test_weights_that_attention_touches(d, heads, m, t, batch, kind):
    assert touch_plan(d, heads, m, t, batch).kind == kind
    assert touch_plan(d, heads, m, t, batch, param_dtype=binding.EP_F32).kind == TOUCH_NONE


# a group of micro-batches uses the K ranges of each, so that other tiles run than for one batch of as many images
@pytest.mark.parametrize("micro,count,group,alone", [(8, 6, TOUCH_NONE, TOUCH_ALL), (9, 3, TOUCH_ALL, TOUCH_NONE)])
def test_weights_that_attention_touches_for_a_group(micro, count, group, alone):
    assert touch_plan(1024, 16, 4096, 197, micro * count, ranges_of=micro).kind == group
    assert touch_plan(1024, 16, 4096, 197, micro * count).kind == alone


# the range holds the weights that it is for, and ends with them: inside the layer where no other follows
@pytest.mark.parametrize("d,heads,m,t,batch", [(64, 1, 64, 15, 1), (192, 3, 768, 197, 4), (768, 12, 3072, 197, 8), (832, 13, 3328, 50, 16),
                                               (1024, 16, 4096, 197, 8), (1024, 16, 4096, 197, 16), (1024, 16, 4096, 197, 1)])
@pytest.mark.parametrize("next_layer", [False, True])
def test_range_of_touched_weights(d, heads, m, t, batch, next_layer):
    p = touch_plan(d, heads, m, t, batch, next_layer=next_layer)
    qkv, proj, fc1, fc2 = zip(p.weights, p.weight_ends)
    for (begin, end), size in zip((qkv, proj, fc1, fc2), (3 * d * d, d * d, d * m, d * m)):
        assert 0 <= begin and end - begin == 2 * size and end <= p.layer_bytes
    inside = {TOUCH_NONE: [], TOUCH_LONG: [proj, fc2], TOUCH_ALL: [proj, fc2, fc1]}[p.kind]
    if p.kind == TOUCH_ALL and next_layer:
        inside.append((p.layer_bytes + qkv[0], p.layer_bytes + qkv[1]))
    assert p.begin == proj[0] and p.end == max([e for _, e in inside], default=p.begin)
    assert all(p.begin <= b for b, _ in inside) and (next_layer or p.end <= p.layer_bytes)
    assert (1 << 30) > p.end - p.begin                                   # offsets of touched lines are 32-bit
