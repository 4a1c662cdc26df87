"""Host logic of the library that needs no GPU: the shape -> kernel dispatcher, the variant
table and the workspace sizing."""
import pytest

from paper_2509_01229_amd import api
from paper_2509_01229_amd import workloads as WL


def _pick(M, N, K, g=64):
    return api.w4a8_variant_name(api.w4a8_select_variant(M, N, K, g))


def _pt_fits(M, N, K):
    return K % 512 == 0 and (M % 128 == 0 or M % 128 > 64)


def _solo_form(M, N, K):
    """The dispatcher's cost rule for the 256-row tiles, restated: costs fitted to measurements, in
    units of a round of 256 tiles of 128 x 256; 1 = 256 x 256 tiles, 2 = 256 x 128 tiles with two k
    groups, 0 = neither."""
    if K % 512:
        return 0
    bm = -(-M // 256)
    t256, t2, t128 = bm * -(-N // 256), bm * -(-N // 128), -(-M // 128) * -(-N // 256)
    def part(t):
        fill = t / 256
        return 0.0 if t == 0 else 0.24 + 0.90 * fill if t <= 128 else 0.47 + 0.52 * fill if t <= 256 else 0.80 + 0.51 * fill
    duo = 2.0 * (t128 // 512) + part(t128 % 512)
    short_k = 1.0 if K >= 4096 else 1.06
    solo = (0.734 + 0.94 * t256 / 256 if t256 <= 256 else 2.0 * -(-t256 // 256) * 0.86) * short_k * 0.92
    g2 = (0.406 + 0.56 * t2 / 256) * short_k if 136 < t2 <= 256 else 1e30
    if solo < duo and solo <= g2:
        return 1
    return 2 if g2 < duo else 0


def test_dispatcher_families_on_the_workloads():
    for s in WL.ALL_SHAPES:
        name = _pick(s.M, s.N, s.K, s.group)
        if s.M <= 16:
            assert name.startswith("stream16_"), (s.name, name)
        elif s.M <= 32:
            assert name == "stream_m32", (s.name, name)
        elif s.M <= 64 and s.N <= 16384:
            assert name == "stream_m64", (s.name, name)
        else:
            assert name in ("duo_m64", "duo_m128", "duo_dl_m128", "duo_pt_m128", "solo16_pt_m256", "solo16_g2_m256",
                            "solo16_g2_sk_m256"), (s.name, name)
            tiles128 = -(-s.M // 128) * -(-s.N // 256)
            form = _solo_form(s.M, s.N, s.K)
            if name == "solo16_g2_sk_m256":   # K slices across blocks: very long K, one round of 256 x 128 tiles x slices
                assert not form and s.K >= 16384 and -(-s.M // 256) * -(-s.N // 128) <= 128, (s.name, name)
            elif form:                  # 256-row tiles, one wave per SIMD, where their whole rounds come out ahead
                assert name == ("solo16_pt_m256" if form == 1 else "solo16_g2_m256"), (s.name, name)
            elif tiles128 > 256:      # more tiles than CUs: the direct-to-LDS pipeline, persistent where it fits
                assert name == ("duo_pt_m128" if _pt_fits(s.M, s.N, s.K) else "duo_dl_m128"), (s.name, name)
            elif tiles128 > 128 and s.K % 512 == 0:   # more than half a round: persistent, one block per CU
                assert name == "duo_pt_m128", (s.name, name)
            elif -(-s.M // 64) * -(-s.N // 256) > 256:
                assert name == "duo_m128", (s.name, name)
        v = api.w4a8_select_variant(s.M, s.N, s.K, s.group)
        assert api.w4a8_variant_supports(v, s.M, s.N, s.K, s.group)


def test_dispatcher_boundaries():
    assert _pick(8, 4096, 4096) == "stream16_f1_w16_s1"        # short K: sixteen waves per block, one tile
    assert _pick(16, 4096, 4096) == "stream16_f1_w16_s1" and _pick(16, 4096, 2048) == "stream16_f1_w16_s1"
    assert _pick(8, 8192, 8192) == "stream16_f1_w8_u4"         # K to 8192: deep prefetch, whole K in the block
    assert _pick(16, 8192, 8192) == "stream16_f1_w16_s1" and _pick(16, 4096, 8192) == "stream16_f1_w8"
    assert _pick(16, 4096, 11008) == "stream16_f1_w8"          # longer K: K slices across blocks
    assert _pick(16, 8192, 28672, 128) == "stream16_f2_w8"     # 129..256 tiles, long K: two tiles per block
    assert _pick(4, 8192, 28672, 128) == "stream16_f1_w16_s1"  # ... up to 8 rows: sixteen waves split K
    assert _pick(4, 4096, 16384) == "stream16_f1_w8" and _pick(16, 8192, 14336) == "stream16_f1_w8"
    assert _pick(16, 11008, 4096) == "stream16_f2_w16_s1"      # more than 256 tiles: two per block
    assert _pick(4, 16384, 4096) == "stream16_f1_w16_s1" and _pick(16, 16384, 8192) == "stream16_f2_w8"
    assert _pick(16, 28672, 2048) == "stream16_f2_w8"
    assert _pick(16, 28672, 8192, 128) == "stream16_f2_w4"     # N alone fills the chip
    assert _pick(17, 4096, 4096) == "stream_m32" and _pick(32, 28672, 8192) == "stream_m32"
    assert _pick(33, 4096, 4096) == "stream_m64" and _pick(64, 16384, 4096) == "stream_m64"
    # 33..64 rows: streamed (X through LDS) up to 512 tiles of 32 channels, whatever K
    assert _pick(64, 8192, 8192) == "stream_m64" and _pick(48, 8192, 8192) == "stream_m64"
    assert _pick(40, 8192, 28672, 128) == "stream_m64" and _pick(64, 4096, 11008) == "stream_m64"
    # ... except 129..256 tiles with very long K from 48 rows on: the tiles' split-K grid
    assert _pick(64, 8192, 28672, 128) in ("duo_m64", "duo_m128") and _pick(48, 6144, 28672, 128) in ("duo_m64", "duo_m128")
    assert _pick(64, 4096, 28672, 128) == "stream_m64" and _pick(64, 8192, 16384, 128) == "stream_m64"
    assert _pick(64, 28672, 8192) == "duo_m64" and _pick(65, 4096, 4096) == "duo_m64"
    assert _pick(256, 28672, 8192) == "solo16_g2_m256"           # 224 tiles of 256 x 128: one round, 62 against 66 us
    assert _pick(192, 28672, 8192) == "solo16_g2_m256" and _pick(128, 28672, 8192) == "duo_m128"
    assert _pick(512, 4096, 4096) == "duo_m64" and _pick(1025, 4096, 4096) == "solo16_g2_m256"
    # very long K, nearly full 256-row tiles: the 256 x 128 tiles with K slices across blocks
    assert _pick(256, 8192, 28672, 128) == "solo16_g2_sk_m256" and _pick(512, 8192, 28672, 128) == "solo16_g2_sk_m256"
    assert _pick(256, 6144, 16384, 128) == "solo16_g2_sk_m256" and _pick(250, 8192, 16384) == "solo16_g2_sk_m256"
    assert _pick(256, 4096, 16384, 128) == "duo_m64"           # (four slices of 32 tiles: half a round)
    assert _pick(128, 8192, 28672, 128) in ("duo_m64", "duo_m128") and _pick(384, 8192, 28672, 128) == "duo_m128"
    assert _pick(256, 8192, 14336, 128) in ("duo_m64", "duo_m128")
    assert _pick(256, 8192, 8192) == "duo_m64" and _pick(256, 10240, 8192, 128) == "duo_m128"
    assert _pick(128, 4096, 256) == "duo_m128"                 # one k unit: no room for two k groups
    # 256-row tiles, one wave per SIMD: 256 x 128 as one round on more than half of the CUs ...
    assert _pick(1024, 8192, 8192) == "solo16_g2_m256" and _pick(960, 8192, 8192) == "solo16_g2_m256"
    assert _pick(2048, 4096, 11264) == "solo16_g2_m256"
    assert _pick(768, 8192, 8192) == "solo16_g2_m256"            # 192 tiles: 54 against 58 us
    assert _pick(512, 9216, 8192) == "solo16_g2_m256" and _pick(512, 11008, 4096) == "solo16_g2_m256"   # 144 / 172 tiles
    assert _pick(512, 10240, 2048) in ("solo16_g2_m256", "duo_pt_m128") and _pick(1024, 5120, 8192) == "solo16_g2_m256"
    assert _pick(512, 8192, 8192) == "duo_m128" and _pick(1024, 4096, 8192) in ("duo_m64", "duo_m128")   # 128 tiles: equal or behind
    assert _pick(384, 8192, 8192) == "duo_m128"                # (a third of the second row tile's work is lost)
    # ... 256 x 256 where their whole rounds cost less than the rounds of 128-row tiles, two blocks to a CU
    assert _pick(1152, 8192, 8192) == "solo16_pt_m256" and _pick(1280, 8192, 8192) == "solo16_pt_m256"   # 160 tiles, one round
    assert _pick(4096, 8192, 8192) == "solo16_pt_m256" and _pick(2048, 8192, 28672, 128) == "solo16_pt_m256"
    assert _pick(8192, 8192, 8192) == "solo16_pt_m256" and _pick(4096, 8192, 2048) == "solo16_pt_m256"
    assert _pick(1024, 28672, 8192, 128) == "solo16_pt_m256" and _pick(2048, 28672, 8192, 128) == "solo16_pt_m256"
    assert _pick(1024, 10240, 8192, 128) == "solo16_pt_m256" and _pick(1024, 11008, 4096) == "solo16_pt_m256"
    # ... and the 128-row tiles where a last round of 256-row tiles would be mostly empty
    assert _pick(2560, 8192, 8192) == "duo_pt_m128" and _pick(3072, 8192, 8192) == "duo_pt_m128"
    assert _pick(2048, 10240, 8192, 128) == "duo_pt_m128" and _pick(2048, 11008, 4096) == "duo_pt_m128"
    # K % 512 == 256: the 16x16x64 forms of the 256-row tiles take it (two added stages of zero weights),
    # the persistent 128-row tiles do not
    assert _pick(4096, 8192, 11008) == "solo16_pt_m256" and _pick(4096, 4096, 11008) == "solo16_pt_m256"
    assert _pick(2048, 4096, 11008) == "solo16_g2_m256" and _pick(2560, 8192, 11008) == "duo_dl_m128"
    assert _pick(4096 + 40, 8192, 8192) == "duo_dl_m128"       # (rounds of 256-row tiles: 3 against 2.06) ragged last row tile of at most 64 rows: its two-fragment path
    assert _pick(4096 + 100, 8192, 8192) == "duo_pt_m128"
    with pytest.raises(api.LiquidGemmError):
        api.w4a8_select_variant(8, 100, 512, 64)                # bad shape


def _plan(M, N, K, g=64):
    return [(rows, api.w4a8_variant_name(v)) for rows, v in api.w4a8_select_plan(M, N, K, g)]


def test_two_launch_plans():
    """Batches whose 256 x 256 tiles make whole rounds of the chip plus a rest of at most 256 rows,
    or a larger rest that does not take 256 x 256 tiles itself, run as two launches over consecutive
    rows where the cost rule says so; everything else as one, which is then the dispatcher's choice."""
    assert _plan(4096 + 40, 8192, 8192) == [(4096, "solo16_pt_m256"), (40, "stream_m64")]      # a ragged tail of the batch
    assert _plan(2048 + 100, 8192, 4096) == [(2048, "solo16_pt_m256"), (100, "duo_m64")]
    assert _plan(1024 + 30, 16384, 4096, 128) == [(1024, "solo16_pt_m256"), (30, "stream_m32")]
    # larger rests that fill most of a round of 256 x 128 tiles (143 against 150 us, 157 against 162, 240 against 255)
    assert _plan(2048, 10240, 8192, 128) == [(1536, "solo16_pt_m256"), (512, "solo16_g2_m256")]
    assert _plan(3072, 8192, 8192) == [(2048, "solo16_pt_m256"), (1024, "solo16_g2_m256")]
    assert _plan(1280, 28672, 8192, 128) == [(1024, "solo16_pt_m256"), (256, "solo16_g2_m256")]
    assert _plan(2748, 8192, 4096) == [(2048, "solo16_pt_m256"), (700, "solo16_g2_m256")]
    # ... also a rest on 128-row tiles (143 against 156 us, 423 against 513)
    assert _plan(2560, 8192, 8192) == [(2048, "solo16_pt_m256"), (512, "duo_m128")]
    assert _plan(2560, 8192, 28672, 128) == [(2048, "solo16_pt_m256"), (512, "solo16_g2_sk_m256")]
    # ... but not a rest that would be 256 x 256 tiles again, nor with short K
    assert _plan(3584, 8192, 8192) == [(3584, "solo16_pt_m256")] and _plan(2304, 11008, 4096) == [(2304, "solo16_pt_m256")]
    assert _plan(2748, 8192, 512) == [(2748, _pick(2748, 8192, 512))]
    # K % 512 == 256 splits like any other K (the 16x16x64 forms take it)
    assert _plan(3072, 8192, 8448) == [(2048, "solo16_pt_m256"), (1024, "solo16_g2_m256")]
    for M, N, K, g in [(4096, 8192, 8192, 64), (2048, 28672, 8192, 128), (1536, 8192, 8192, 64), (16, 8192, 8192, 64),
                       (256, 8192, 8192, 64), (2048, 11008, 4096, 64), (0, 4096, 4096, 64)]:
        assert _plan(M, N, K, g) == [(M, _pick(M, N, K, g))], (M, N, K)
    for s in WL.ALL_SHAPES:
        plan = api.w4a8_select_plan(s.M, s.N, s.K, s.group)
        assert sum(rows for rows, _ in plan) == s.M and all(rows > 0 for rows, _ in plan)
        assert all(api.w4a8_variant_supports(v, rows, s.N, s.K, s.group) for rows, v in plan)
        assert len(plan) == 1 or plan[0][0] % 256 == 0


def test_variant_table_is_consistent():
    names = api.w4a8_variant_names()
    assert len(names) == len(set(names)) == api.w4a8_variant_count()
    for v, name in enumerate(names):
        # row limits are part of the names' families
        limit = (16 if name.startswith("stream16") else 64 if name.startswith("stream_m64")
                 else 32 if name.startswith(("stream_f", "stream_x_", "stream_m32"))
                 else 256 if name in ("solo16_pt_m256_s2", "solo16_g2_m256_s4") else None)
        if limit:
            assert api.w4a8_variant_supports(v, limit, 256, 2048, 64)
            assert not api.w4a8_variant_supports(v, limit + 1, 256, 2048, 64)
        else:
            assert api.w4a8_variant_supports(v, 4096, 256, 1024, 64)
        assert not api.w4a8_variant_supports(v, 8, 96, 1024, 64)   # N % 64 != 0
        assert not api.w4a8_variant_supports(v, 8, (1 << 26) + 64, 1024, 64)   # rows addressed in 32 bits
        assert not api.w4a8_variant_supports(v, 8, 256, 131072 + 256, 64)      # the accumulator's range
    assert not api.w4a8_variant_supports(-1, 8, 256, 1024, 64)
    assert not api.w4a8_variant_supports(len(names), 8, 256, 1024, 64)


def test_reported_kernels():
    """What w4a8_describe_launch says runs: a named variant is the kernel of that name (stream_m32 and
    stream_m64 stand for panel forms); the dispatcher takes tiles or a panel where the plan says duo_m64 or duo_m128."""
    names = api.w4a8_variant_names()
    for M, N, K in [(8, 256, 512), (77, 448, 768), (200, 256, 512), (130, 576, 1280), (300, 320, 1792), (256, 8192, 8192),
                    (160, 512, 2048), (200, 1024, 4096)]:
        for v, name in enumerate(names):
            if api.w4a8_variant_supports(v, M, N, K, 64) and name not in ("stream_m32", "stream_m64"):
                assert api.w4a8_describe_launch(M, N, K, 64, v)[0] == name
    assert api.w4a8_describe_launch(45, 4096, 4096, 64, names.index("stream_m64"))[0].startswith("panel_f")
    with pytest.raises(api.LiquidGemmError):
        api.w4a8_describe_launch(65, 4096, 4096, 64, names.index("stream_m64"))
    with pytest.raises(api.LiquidGemmError):
        api.w4a8_describe_launch(8, 100, 512, 64)
    # both are duo_m64 to w4a8_select_variant
    assert _pick(256, 8192, 8192) == _pick(64, 28672, 8192) == "duo_m64"
    assert api.w4a8_describe_launch(256, 8192, 8192, 64) == ("panel_f4_m64", 0)
    assert api.w4a8_describe_launch(64, 28672, 8192, 64) == ("panel_f4_m64", 0)
    assert api.w4a8_describe_launch(34, 25536, 1792, 64) == ("duo_m64", 32768 + 100 * 2 * 131072)   # two K slices
    assert api.w4a8_describe_launch(64, 1088, 6912, 64)[0] == "panel_f1_m32_s3"
    assert api.w4a8_describe_launch(4096 + 40, 8192, 8192, 64)[0] == "solo16_pt_m256[4096 rows]+panel_f2_m32[40 rows]"
    assert api.w4a8_describe_launch(0, 8192, 8192, 64) == ("", 0)
    for s in WL.ALL_SHAPES:
        name, _ = api.w4a8_describe_launch(s.M, s.N, s.K, s.group)
        plan = api.w4a8_select_plan(s.M, s.N, s.K, s.group)
        for part, (rows, v) in zip(name.split("+"), plan):
            picked = names[v]
            assert part.split("[")[0] == picked or (picked in ("duo_m64", "duo_m128", "stream_m32", "stream_m64")
                                                    and part.startswith("panel_f")), (s.name, name)


def test_workspace_sizes():
    ws = api.w4a8_gemm_workspace_size
    assert ws(0, 4096, 4096, 64) == 0 and ws(16, 100, 4096, 64) == 0     # nothing to do / bad shape
    assert ws(4096, 8192, 8192, 64) == 0                                  # enough tiles: no split-K
    small = ws(16, 4096, 4096, 64)
    assert small > 0 and small % 16 == 0
    # room for 16 slices of the 16-row kernels' partial tiles at least
    assert small >= 16 * (4096 // 32) * 8 * 64 * 4
    # the tiled kernel's partial tiles (128 x 256 INT32 per tile and slice, up to 8 slices)
    assert ws(128, 4096, 4096, 64) >= 16 * 8 * 128 * 256 * 4
    assert ws(128, 4096, 4096, 64) <= 1 << 30


def test_workspace_size_covers_what_it_promises():
    """w4a8_gemm_workspace_size is enough for the dispatcher, for the variants of up to 256 rows and, on fewer than
    192 tiles of 128 x 256, for every variant that can run the shape."""
    names = api.w4a8_variant_names()
    shapes = [(M, N, K) for M in (1, 16, 17, 32, 33, 64, 65, 128, 257, 512, 1000, 2048, 4096, 12000)
              for N in (64, 192, 256, 1536, 4096, 8192, 28672, 65600) for K in (256, 512, 768, 1024, 2048, 8192, 28672)]
    for M, N, K in shapes:
        room = api.w4a8_gemm_workspace_size(M, N, K, 64)
        few_tiles = -(-M // 128) * -(-N // 256) < 192
        for v in range(-1, len(names)):
            if v >= 0 and not api.w4a8_variant_supports(v, M, N, K, 64):
                continue
            if v >= 0 and not few_tiles and api.w4a8_variant_supports(v, 4096, N, 2048, 64):
                continue   # (no row limit: may name K slices of a larger output)
            name, need = api.w4a8_describe_launch(M, N, K, 64, v)
            if "+" in name:
                continue   # (the rest of a batch in two launches takes the slices that fit)
            assert need <= room, (M, N, K, names[v] if v >= 0 else name, need, room)
    # what it points to for the others
    v = names.index("panel_f4_m32_s2")
    assert api.w4a8_describe_launch(2048, 8192, 512, 64, v)[1] == 32768 + 64 * 64 * 2 * 4 * 4096
    assert api.w4a8_gemm_workspace_size(2048, 8192, 512, 64) < 32768 + 64 * 64 * 2 * 4 * 4096


def test_workload_names():
    # the listed shapes by name, and any other shape spelled <label>_M.._N.._K..[_g..]
    s = WL.by_name("l70b_up_M16_N28672_K8192")
    assert (s.M, s.N, s.K, s.group) == (16, 28672, 8192, 128)
    s = WL.by_name("curve_M64_N8192_K8192_g128")
    assert (s.M, s.N, s.K, s.group) == (64, 8192, 8192, 128)
    assert WL.by_name("x_M3_N64_K256").group == 64
    for bad in ("bogus", "x_M3_N64", "x_M3_N64_K256_g32", "_M3_N64_K256"):
        with pytest.raises(KeyError):
            WL.by_name(bad)


def test_panels_of_several_rounds():
    """32 x 128 panels run one on a CU: beyond one round of them 32 x 64 panels take their place (15.9 against 13.1
    us); so they do for 32 x 32 panels of more than two rounds while K is short (5.5 against 5.2 us)."""
    name = lambda M, N, K, g: api.w4a8_describe_launch(M, N, K, g)[0]
    for g in (64, 128):
        assert name(136, 11520, 2048, g) == name(160, 11520, 2048, g) == name(136, 13056, 3072, g) == "panel_f2_m32"
        assert name(28, 24576, 3584, g) == "panel_f4_m32"   # one round
        for K in (256, 512, 768):
            assert name(24, 24064, K, g) == "panel_f2_m32" and name(24, 8192, K, g) == "panel_f1_m32"
        assert name(24, 24064, 1024, g) == "panel_f1_m32"


def test_panels_instead_of_few_tiles_by_estimate_alone():
    """33 to 512 rows: panels where they are estimated to be clearly faster than few tiles, for both group sizes alike and
    for every number of channels and rows (20000 calls that kept the tiles: 0.83 of the time on panels)."""
    import random

    name = lambda M, N, K, g: api.w4a8_describe_launch(M, N, K, g)[0]
    rng = random.Random(4)
    for _ in range(3000):
        M, N, K = rng.randint(33, 512), 64 * rng.randint(16, 512), 256 * rng.randint(8, 64)
        assert name(M, N, K, 64) == name(M, N, K, 128), (M, N, K)
    for g in (64, 128):
        for N in (10176, 10240, 12672, 12736):
            assert name(70, N, 2304, g).startswith("panel_f") and name(100, N, 2304, g).startswith("panel_f"), N
        for M in (62, 63, 64):
            assert name(M, 28672, 2048, g) == name(M, 28672, 8192, g) == name(M, 30720, 4352, g) == "panel_f4_m64", M
        assert name(256, 10240, 8192, g) == "panel_f3_m128" and name(130, 12352, 5376, g) == "panel_f2_m32"


def test_four_slices_of_wide_panels_with_very_long_k():
    """Two K slices of 32 x 64 panels stand in for four of 32 x 128 up to K = 40960 and are behind them beyond 49152."""
    name = lambda M, N, K, g: api.w4a8_describe_launch(M, N, K, g)[0]
    for g in (64, 128):
        for M, N in ((88, 2432), (32, 5952), (32, 7040)):
            assert name(M, N, 40960, g) == "panel_f2_m32_s2" and name(M, N, 114688, g) == name(M, N, 65536, g) == "panel_f4_m32_s4"


def test_where_half_tiles_and_panels_are_behind_whole_tiles():
    """Up to 16 rows whole tiles stay where they were found ahead: K below 2048, 9 and 10 rows on 129..256 tiles with
    all of a wave's loads in flight, K slices of half tiles for more than 10 rows of up to 16 tiles."""
    def runs(M, N, K):
        name = api.w4a8_describe_launch(M, N, K, 64)[0]
        return name.split("[as ")[1][:-1] if "[as " in name else None

    for M in (1, 4, 9, 16):
        assert [runs(M, N, K) for N in (64, 2048, 4096) for K in (256, 512, 1024, 1536, 1792)] == [None] * 15
        assert runs(M, 64, 2048) == runs(M, 4096, 2048) == "stream16_h_w8_d2"
    for M in (9, 10):
        assert runs(M, 7360, 7168) is None and runs(M, 8192, 8192) is None and runs(M, 7360, 7424) == "panel_f1_m32"
    assert runs(11, 7360, 7168) == runs(9, 7360, 8448) == "panel_f1_m32"
    assert runs(12, 512, 8448) is None and runs(11, 512, 12544) is None
    assert runs(10, 512, 8448) == runs(12, 576, 8448) == "stream16_h_w8_d3_s2"
    assert runs(10, 512, 12544) == runs(12, 576, 12544) == "stream16_h_w8_d4_s2"


def test_two_tile_blocks_of_eight_waves_keep_k_up_to_2048():
    """769..896 tiles from 9 rows on: panels for K from 2304 on, where these blocks have four waves."""
    runs = lambda M, N, K, g: api.w4a8_describe_launch(M, N, K, g)[0]
    for g in (64, 128):
        for M, N in ((9, 24640), (16, 28672)):
            assert runs(M, N, 2048, g) == "stream16_f2_w8" and runs(M, N, 2304, g) == "stream16_f2_w4[as panel_f2_m32]"
        assert runs(8, 28672, 2048, g) == "stream16_f2_w8[as stream16_f1_w8]"


def test_half_tiles_of_8_rows_end_at_very_long_k():
    """Up to 128 tiles with K beyond 49152: 7 rows are ahead on half tiles, 8 rows on whole ones."""
    runs = lambda M, N, K, g: api.w4a8_describe_launch(M, N, K, g)[0]
    for g in (64, 128):
        for N, form in ((1344, "stream16_h_w8_d2_s2"), (4032, "stream16_h_w8_d2")):
            for M, K in ((8, 49152), (7, 49408), (7, 129536), (1, 131072)):
                assert runs(M, N, K, g).endswith(f"[as {form}]"), (M, N, K)
            for K in (49408, 66048, 129536):
                assert runs(8, N, K, g) == "stream16_f1_w8", (N, K)


def test_up_to_8_rows_of_one_tile_a_block_go_by_ranges_of_k():
    """129..256 tiles: sixteen waves of one tile, half tiles where their passes are full or nearly so; no single K is an exception."""
    runs = lambda M, N, K, g: api.w4a8_describe_launch(M, N, K, g)[0].split("[as ")[-1].rstrip("]")
    for g in (64, 128):
        for N in (4160, 8192):
            for M in (1, 4, 5, 8):
                assert {runs(M, N, K, g) for K in range(8448, 12288, 256)} == {"stream16_f1_w16_s1"}
                assert {runs(M, N, K, g) for K in (5888, 6144)} == {"stream16_h_w8_d3"}
                assert {runs(M, N, K, g) for K in (4352, 5632, 6400, 7680)} == {"stream16_f1_w16_s1"}
                assert {runs(M, N, K, g) for K in (7936, 8192)} == {"stream16_h_w8_d4" if M <= 4 else "stream16_f1_w16_s1"}


def _grouped(rows, N, K, g):
    offsets = [0]
    for r in rows:
        offsets.append(offsets[-1] + r)
    return api.w4a8_describe_grouped(offsets, N, K, g)


def test_reported_grouped_launches():
    """What w4a8_describe_grouped says a grouped call launches: every row exactly once, at most five launches."""
    import re

    assert _grouped([0, 0], 256, 512, 64) == ""
    assert _grouped([3, 0, 16], 256, 512, 64) == "stream16_f2_w8[2 experts, 19 rows]"
    assert _grouped([17, 32, 0, 1], 256, 512, 64) == "panel_f2_m32[3 experts, 50 rows]"
    assert _grouped([40, 64, 9], 4096, 4096, 64) == "panel_f4_m64[3 experts, 113 rows]"
    assert _grouped([760, 741, 768, 733, 742, 789, 722, 745], 4096, 14336, 64).startswith("solo16_")
    for rows, N, K, g in [([1500, 20, 1537, 1400, 1700, 7], 4096, 4096, 64), ([1] * 64, 2816, 256, 128), ([129, 128, 127, 33, 257], 64, 256, 64),
                          ([700, 5, 520, 900, 40, 256, 1000], 4160, 768, 128), ([90, 100, 3, 17, 65], 8192, 1024, 64)]:
        parts = [re.fullmatch(r"([a-z0-9_]+)\[(\d+) experts, (\d+) rows\]", part) for part in _grouped(rows, N, K, g).split("+")]
        assert all(parts) and len(parts) <= 5 and len({p[1] for p in parts}) == len(parts)
        assert sum(int(p[3]) for p in parts) == sum(rows)
    for E, offsets, N, K, g in [(2, [0, 3, 2], 256, 512, 64), (1, [1, 4], 256, 512, 64), (1, [0, 4], 100, 512, 64), (1, [0, 4], 256, 512, 32)]:
        with pytest.raises(api.LiquidGemmError):
            api.w4a8_describe_grouped(offsets, N, K, g)


def test_grouped_rules():
    """Large experts: what the single GEMMs' rule picks unless another split is estimated to be clearly faster.  With
    short K the 128-row tiles' estimate is too low: they were picked where 256 x 256 tiles took three quarters of the time."""
    # 256 x 256 tiles with short K (121 us on 128-row tiles, 90 on these), and 128-row tiles where K % 512 == 256 adds two stages
    for rows, N, K, g in [([3648, 3671], 15936, 512, 128), ([511, 620, 909, 5716], 16320, 512, 128), ([2113, 2153], 16320, 1024, 64),
                          ([746, 761, 797, 819], 16192, 1024, 128)]:
        assert _grouped(rows, N, K, g).startswith("solo16_pt_m256["), (rows, N, K)
    assert _grouped([3648, 3671], 15936, 768, 128).startswith("duo_dl_m128[")
    # 24 row blocks on 16 column blocks of 256: one and a half rounds
    assert _grouped([760, 741, 768, 733, 742, 789, 722, 745], 4096, 14336, 64).startswith("solo16_pt_m256[6 experts, 4000 rows]+solo16_g2_m256[")
    # two kinds of 256-row tiles only where they are far ahead (115 us on 128-row tiles, 131 on two kinds; 129 and 147; 215 and 246)
    for rows, N, K, g in [([1324], 16128, 5376, 64), ([933, 304, 1067, 1181], 5696, 6144, 128), ([1118, 1138, 1162, 1131], 8256, 6144, 128)]:
        assert _grouped(rows, N, K, g).startswith("duo_dl_m128["), (rows, N, K)
    # 64-row panels of 128 channels, one on a CU: not a little beyond a round of them (38 us on tiles, 47 on panels; 51 and 62)
    assert _grouped([69, 52, 57, 57, 46, 63, 58, 59, 49, 43, 55, 48, 60, 48, 64, 45], 2176, 6656, 64).startswith("duo_m64[16")
    assert _grouped([75, 63], 13056, 9984, 64).startswith("duo_m64[2")
    # short K (7.9 us on tiles, 8.8 on panels), and where panels are far ahead (55.8 us on tiles, 19.4)
    assert _grouped([75, 63, 77, 75], 4672, 256, 64).startswith("duo_m128")
    assert _grouped([128], 4096, 14336, 64) == "panel_f2_m32[1 experts, 128 rows]"


def test_a_failed_launch_names_the_kernel_that_ran():
    """Without a GPU every launch fails; the error names the kernel that was launched, not the one it stands for."""
    import ctypes

    import torch

    if torch.cuda.is_available():
        pytest.skip("the launches have to fail")
    buf = ctypes.create_string_buffer(4096 + 16)
    p = ctypes.c_void_p((ctypes.addressof(buf) + 15) // 16 * 16)   # (never read: nothing is launched)
    for M, N, K, name in [(4, 4096, 4096, "stream16_h_w8_d2"), (4, 4096, 11008, "stream16_h_w16_d3"), (4, 4096, 1024, "stream16_f1_w16_s1")]:
        with pytest.raises(api.LiquidGemmError, match=f"launch of {name} failed"):
            api._check(api.lib().w4a8_gemm(M, N, K, 64, p, p, p, p, p, p, None, 0, None))
