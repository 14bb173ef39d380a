"""Per-kernel parity: each HIP kernel, called through the C ABI's single-operation entry
points, against the CPU oracle fed the same bf16-rounded inputs.

Tolerances (max |gpu - ref| / max |ref| over the compared tensor):
  fp32 accumulator outputs  <= 1e-3   (inputs identical; only summation order differs)
  bf16 outputs              <= 2e-2   (one or two bf16 roundings on the way out)
"""
import numpy as np
import pytest

from oracle import transformer as T
from paper_2504_19516_amd import synth

pytestmark = pytest.mark.gpu

ACC_TOL, BF16_TOL = 1e-3, 2e-2


def rel(a, b):
    return float(np.abs(np.asarray(a, np.float64) - np.asarray(b, np.float64)).max() / np.abs(b).max())


@pytest.fixture(scope="module")
def sts():
    from paper_2504_19516_amd import sts as m
    m.lib()
    return m


@pytest.mark.parametrize("cfg,m", [("256x256", 300), ("128x128", 300), ("64x256", 70), ("64x256", 20), ("64x128", 64), ("128x128", 1),
                                   ("64x128", 50), ("256x256", 513), ("128x256", 129), ("128x256", 300)])
def test_gemm_fp32_accumulators(sts, cfg, m):
    n, k = 512, 320
    a = synth.normal_bf16(1, (m, k))
    w = synth.normal_bf16(2, (n, k), 0.05)
    ref = T.op_linear(a.astype(np.float64), w.astype(np.float64))
    got = sts.op_gemm(a, w, cfg, epilogue=1)
    assert rel(got, ref) <= ACC_TOL
    assert rel(got, ref) <= 1e-5          # in practice fp32 accumulation of 320 terms


@pytest.mark.parametrize("cfg", ["256x256", "128x128", "64x128", "64x256", "128x256"])
@pytest.mark.parametrize("k", [64, 128, 192, 576])
@pytest.mark.parametrize("epilogue", [0, 1])
def test_gemm_short_and_odd_k_extents(sts, cfg, k, epilogue):
    """One, two, three and nine K tiles: the prologue, the steady loop and the surplus loads of the last iterations of every
    main loop (the 256x256 loop keeps three activation stages and requests operands a tile ahead), rows that end inside a tile."""
    m, n = 290, 512
    a = synth.normal_bf16(11, (m, k))
    w = synth.normal_bf16(12, (n, k), 0.1)
    ref = T.op_linear(a.astype(np.float64), w.astype(np.float64))
    got = sts.op_gemm(a, w, cfg, epilogue=epilogue)
    assert rel(got, ref) <= (BF16_TOL if epilogue == 0 else 1e-5)


@pytest.mark.parametrize("cfg,m,split", [("64x256", 64, 4), ("64x256", 8, 8), ("128x128", 130, 2), ("64x128", 33, 3), ("64x128", 64, 8),
                                         ("256x256", 300, 2), ("128x256", 200, 4)])
def test_gemm_split_k(sts, cfg, m, split):
    n, k = 256, 1024
    a = synth.normal_bf16(3, (m, k))
    w = synth.normal_bf16(4, (n, k), 0.05)
    ref = T.op_linear(a.astype(np.float64), w.astype(np.float64))
    assert rel(sts.op_gemm(a, w, cfg, epilogue=1, split_k=split), ref) <= 1e-5


@pytest.mark.parametrize("cfg", ["256x256", "128x128", "64x128", "64x256", "128x256"])
def test_gemm_bf16_store_and_residual(sts, cfg):
    m, n, k = 200, 256, 192
    a = synth.normal_bf16(5, (m, k))
    w = synth.normal_bf16(6, (n, k), 0.05)
    ref = T.op_linear(a.astype(np.float64), w.astype(np.float64))
    got = sts.op_gemm(a, w, cfg, epilogue=0)
    assert rel(got, ref) <= BF16_TOL
    assert np.array_equal(got, synth.to_bf16(got))                   # really bf16 values
    x = np.random.default_rng(7).standard_normal((m, n)).astype(np.float32)
    got2 = sts.op_gemm(a, w, cfg, epilogue=2, c_in=x)
    assert rel(got2, x.astype(np.float64) + ref) <= 1e-5


@pytest.mark.parametrize("cfg,m", [("256x256", 260), ("128x128", 100), ("128x128", 5), ("256x256", 513), ("64x128", 64), ("64x128", 37),
                                   ("64x128", 130)])
def test_gemm_swiglu_epilogue(sts, cfg, m):
    n2, k = 256, 448
    a = synth.normal_bf16(8, (m, k))
    wg = synth.normal_bf16(9, (n2, k), 0.2)
    wu = synth.normal_bf16(10, (n2, k), 0.2)
    a64 = a.astype(np.float64)
    ref = T.silu(T.op_linear(a64, wg.astype(np.float64))) * T.op_linear(a64, wu.astype(np.float64))
    got = sts.op_gemm(a, np.concatenate([wg, wu]), cfg, epilogue=3)
    assert rel(got, ref) <= BF16_TOL


SKINNY = [("64x256s", 256), ("64x320s", 320), ("64x384s", 384), ("64x448s", 448), ("64x512s", 512)]


@pytest.mark.parametrize("cfg,width", SKINNY)
@pytest.mark.parametrize("m,k,split", [(64, 64, 1), (37, 128, 1), (1, 192, 1), (64, 256, 1), (130, 576, 1), (64, 1024, 4), (50, 1088, 3), (8, 2048, 8)])
def test_gemm_skinny_tiles_fp32(sts, cfg, width, m, k, split):
    """The decode tiles (64 rows, 64 columns per wave, weights streamed into registers three K tiles deep): fewer K tiles than
    the pipeline is deep, a K extent that leaves surplus iterations in its last round, rows that end inside a tile and more
    than one tile of rows, slices along K of unequal length."""
    n = 2 * width
    a = synth.normal_bf16(21, (m, k))
    w = synth.normal_bf16(22, (n, k), 0.05)
    ref = T.op_linear(a.astype(np.float64), w.astype(np.float64))
    assert rel(sts.op_gemm(a, w, cfg, epilogue=1, split_k=split), ref) <= 1e-5


@pytest.mark.parametrize("cfg,width", SKINNY)
@pytest.mark.parametrize("m,k", [(64, 448), (29, 128)])
def test_gemm_skinny_tiles_epilogues(sts, cfg, width, m, k):
    n = 2 * width
    a = synth.normal_bf16(23, (m, k))
    a64 = a.astype(np.float64)
    w = synth.normal_bf16(24, (n, k), 0.1)
    ref = T.op_linear(a64, w.astype(np.float64))
    got = sts.op_gemm(a, w, cfg, epilogue=0)
    assert rel(got, ref) <= BF16_TOL and np.array_equal(got, synth.to_bf16(got))
    x = np.random.default_rng(25).standard_normal((m, n)).astype(np.float32)
    assert rel(sts.op_gemm(a, w, cfg, epilogue=2, c_in=x), x.astype(np.float64) + ref) <= 1e-5
    wg, wu = w[:width], w[width:]
    ref3 = T.silu(T.op_linear(a64, wg.astype(np.float64))) * T.op_linear(a64, wu.astype(np.float64))
    assert rel(sts.op_gemm(a, w, cfg, epilogue=3), ref3) <= BF16_TOL


@pytest.mark.parametrize("m", [1, 17, 32, 33, 64, 65, 96, 127, 160, 161, 192, 193, 224, 225, 256])
@pytest.mark.parametrize("k,split", [(64, 1), (192, 2), (320, 1), (832, 3), (1088, 8), (2048, 2)])
def test_gemm_all_rows_form_gives_the_bits_of_the_tiles(sts, m, k, split):
    """Every height, rows that end inside a block, K ranges shorter than what is fetched ahead and not a multiple of it, unequal and fewer
    slices, one and several column tiles. fp32: the bits of 128x128 tiles in the same slices. SwiGLU: their bits where one slice is the
    whole K; else the slices' sums are those of the fp32 form and the result is one rounding of bf16 (2^-8 of the value) and the fp32 error of
    the activation away from it in 64 bits."""
    n = 384
    a = synth.normal_bf16(171, (m, k))
    w = synth.normal_bf16(172, (n, k), 0.05)
    want = sts.op_gemm(a, w, "128x128", epilogue=1, split_k=split)
    assert rel(want, T.op_linear(a.astype(np.float64), w.astype(np.float64))) <= 1e-5
    assert np.array_equal(sts.op_gemm_cols(a, w, 1, split), want)
    got = sts.op_gemm_cols(a, w, 3, split)
    if split == 1:
        assert np.array_equal(got, sts.op_gemm(a, w, "128x128", epilogue=3))
    s64 = want.astype(np.float64)
    ref = T.silu(s64[:, :192]) * s64[:, 192:]
    assert np.all(np.abs(got - ref) <= 2.0 ** -8 * np.abs(ref) + 1e-6 * np.abs(s64[:, 192:]) + 1e-30)


def test_gemm_all_rows_form_refuses(sts):
    for m, rows, k, epilogue, split in ((257, 128, 64, 1, 1), (4, 192, 64, 1, 1), (4, 192, 64, 3, 1), (4, 128, 96, 1, 1), (4, 128, 64, 0, 1), (4, 128, 64, 1, 9), (4, 128, 64, 1, 0)):
        with pytest.raises(sts.StsError) as e:
            sts.op_gemm_cols(np.zeros((m, k), np.float32), np.zeros((rows, k), np.float32), epilogue, split)
        assert e.value.code == sts.EINVAL


@pytest.mark.parametrize("m", [1, 32, 33, 96, 97, 160, 192, 224, 225, 255, 257, 400])
@pytest.mark.parametrize("k,slots", [(64, 0), (192, 0), (320, 0), (1088, 3)])
def test_gemm_row_tile_heights(sts, m, k, slots):
    """The 256-column tile has a loop per height (32 to 256 rows): every height, rows that end inside its last block, K
    extents shorter than the operands' ring and with surplus iterations in its last round, every epilogue, and (slots) the last
    wave of tiles cut along K."""
    n = 512
    a = synth.normal_bf16(71, (m, k))
    a64 = a.astype(np.float64)
    w = synth.normal_bf16(72, (n, k), 0.05)
    ref = T.op_linear(a64, w.astype(np.float64))
    assert rel(sts.op_gemm(a, w, "256x256", epilogue=0, tail_slots=slots), ref) <= BF16_TOL
    assert rel(sts.op_gemm(a, w, "256x256", epilogue=1, tail_slots=slots), ref) <= 1e-5
    x = np.random.default_rng(73).standard_normal((m, n)).astype(np.float32)
    assert rel(sts.op_gemm(a, w, "256x256", epilogue=2, c_in=x, tail_slots=slots), x.astype(np.float64) + ref) <= 1e-5
    ref3 = T.silu(ref[:, :n // 2]) * ref[:, n // 2:]
    assert rel(sts.op_gemm(a, w, "256x256", epilogue=3, tail_slots=slots), ref3) <= BF16_TOL
    if not slots and k > 64:
        assert rel(sts.op_gemm(a, w, "256x256", epilogue=1, split_k=2), ref) <= 1e-5


@pytest.mark.parametrize("m", [65, 96, 97, 129, 200, 225, 256, 300])
@pytest.mark.parametrize("k,split", [(1088, 2), (1600, 3), (1024, 4), (4096, 6), (4096, 8), (640, 1)])
def test_gemm_tiles_give_the_same_bits_for_the_same_slices(sts, m, k, split):
    """Decode batches above 64 rows take 128x128 tiles or 256-column row tiles of any height for the slices the planner decided on: the matrix
    instructions, the order along K and the null tile of an odd number of K tiles must not show in the sums."""
    a, w = synth.normal_bf16(76, (m, k)), synth.normal_bf16(77, (512, k), 0.05)
    want = sts.op_gemm(a, w, "128x128", epilogue=1, split_k=split)
    for cfg in ("256x256", "128x256"):
        assert (sts.op_gemm(a, w, cfg, epilogue=1, split_k=split) == want).all(), cfg
    assert rel(want, T.op_linear(a.astype(np.float64), w.astype(np.float64))) <= 1e-5


def test_gemm_swiglu_is_the_same_in_every_tile(sts):
    """Gates of -100 to 100, each the product of two bf16 numbers (exact in fp32), so that every tile finishes the same sums: whole
    tiles of all shapes and the kernel that adds up the pieces of a cut tile give the same bits, also where exp(-gate) nears the end of fp32
    and the result is as small as 1e-36."""
    m, n, k = 64, 1280, 1088
    gate = np.concatenate([np.linspace(-100, 100, n - 40), np.linspace(-89, -86.5, 40)])
    a, w = np.zeros((m, k), np.float32), np.zeros((2 * n, k), np.float32)
    a[:, 0], a[:, 700] = np.linspace(1.0, 0.985, m), np.linspace(0.5, 2.0, m)
    w[:n, 0], w[n:, 700] = gate, np.linspace(3.0, 4.0, n)
    a, w = synth.to_bf16(a), synth.to_bf16(w)
    want = sts.op_gemm(a, w, "128x128", epilogue=3)
    g64 = a[:, :1].astype(np.float64) * w[:n, 0]
    ref = g64 / (1 + np.exp(-g64)) * (a[:, 700:701].astype(np.float64) * w[n:, 700])
    near = (g64 > -88.6) & (g64 < -87.4)
    assert near.sum() > 100 and (np.abs(want - ref)[near] <= 2.0 ** -8 * np.abs(ref)[near]).all()
    assert rel(want, ref) <= BF16_TOL
    for cfg, slots in [("64x128", 0), ("256x256", 0), ("256x256", 3), ("256x256", 64), ("128x128", 64), ("64x256s", 0), ("64x320s", 0), ("64x512s", 0)]:
        assert np.array_equal(sts.op_gemm(a, w, cfg, epilogue=3, tail_slots=slots), want), (cfg, slots)


@pytest.mark.parametrize("m,k", [(40, 64), (161, 192), (256, 320), (256, 256)])
def test_gemm_row_tiles_keep_infinities_to_their_row(sts, m, k):
    """An odd number of K tiles starts with a null tile of zero operands: it must not meet the activations, an infinity of which
    would make it NaN. One row's only non-zero is an infinity, another holds a NaN; every other row is as without them."""
    n = 256
    a, w = synth.normal_bf16(74, (m, k)), synth.normal_bf16(75, (n, k), 0.05)
    a[3], a[m - 1] = 0.0, 0.0
    clean = sts.op_gemm(a, w, "256x256", epilogue=1)
    a[3, 5], a[m - 1, k - 1] = np.inf, np.nan
    got = sts.op_gemm(a, w, "256x256", epilogue=1)
    assert np.array_equal(got[3], np.where(w[:, 5] > 0, np.inf, -np.inf)) and np.isnan(got[m - 1]).all()
    rest = np.ones(m, bool)
    rest[[3, m - 1]] = False
    assert np.array_equal(got[rest], clean[rest])


@pytest.mark.parametrize("cfg,m,n,slots", [("128x128", 300, 512, 8), ("128x128", 300, 512, 10), ("128x128", 300, 512, 40),
                                           ("128x128", 300, 512, 16), ("256x256", 513, 512, 4), ("256x256", 513, 512, 15),
                                           ("64x128", 64, 640, 4), ("128x256", 300, 768, 7), ("128x256", 513, 512, 8)])
@pytest.mark.parametrize("epilogue", [0, 1, 2, 3])
def test_gemm_tail_wave_split(sts, cfg, m, n, slots, epilogue):
    """The tiles of the last, partly filled wave of workgroups (Section 2.2.1) are cut along K and
    summed by a second kernel: same results as whole tiles, for every epilogue."""
    if epilogue == 3 and cfg == "128x256":
        pytest.skip("the 128x256 tile has no SwiGLU form (it serves the projections with a residual epilogue)")
    k = 1024
    a = synth.normal_bf16(40, (m, k))
    a64 = a.astype(np.float64)
    if epilogue == 3:
        wg = synth.normal_bf16(41, (n // 2, k), 0.05)
        wu = synth.normal_bf16(42, (n // 2, k), 0.05)
        ref = T.silu(T.op_linear(a64, wg.astype(np.float64))) * T.op_linear(a64, wu.astype(np.float64))
        got = sts.op_gemm(a, np.concatenate([wg, wu]), cfg, epilogue=3, tail_slots=slots)
        assert rel(got, ref) <= BF16_TOL
        return
    w = synth.normal_bf16(43, (n, k), 0.05)
    ref = T.op_linear(a64, w.astype(np.float64))
    if epilogue == 2:
        x = np.random.default_rng(44).standard_normal((m, n)).astype(np.float32)
        got = sts.op_gemm(a, w, cfg, epilogue=2, c_in=x, tail_slots=slots)
        assert rel(got, x.astype(np.float64) + ref) <= 1e-5
    else:
        got = sts.op_gemm(a, w, cfg, epilogue=epilogue, tail_slots=slots)
        assert rel(got, ref) <= (BF16_TOL if epilogue == 0 else 1e-5)


def test_gemm_rejects_bad_shapes(sts):
    a = np.zeros((4, 100), np.float32); w = np.zeros((256, 100), np.float32)
    with pytest.raises(sts.StsError) as e:
        sts.op_gemm(a, w, "128x128")          # K not a multiple of 64
    assert e.value.code == sts.EINVAL
    with pytest.raises(sts.StsError):
        sts.op_gemm(np.zeros((4, 64), np.float32), np.zeros((192, 64), np.float32), "256x256")   # N not a multiple of the tile
    with pytest.raises(sts.StsError) as e:
        sts.op_gemm(np.zeros((4, 64), np.float32), np.zeros((512, 64), np.float32), "64x256", epilogue=3)   # no SwiGLU form of this tile
    assert e.value.code == sts.EINVAL
    with pytest.raises(sts.StsError) as e:
        sts.op_gemm(np.zeros((4, 64), np.float32), np.zeros((512, 64), np.float32), "128x256", epilogue=3)  # nor of this one
    assert e.value.code == sts.EINVAL


@pytest.mark.parametrize("t,prior,nq,nkv,d", [(128, 0, 4, 4, 64), (300, 0, 8, 2, 128), (70, 45, 4, 1, 128), (1, 0, 4, 4, 64),
                                              (200, 330, 4, 4, 64), (129, 16, 8, 2, 128),
                                              (130, 16500, 4, 1, 128),      # context beyond one block-table window (16384 tokens)
                                              (40, 33000, 4, 1, 64)])       # ... beyond two
def test_prefill_attention(sts, t, prior, nq, nkv, d):
    q = synth.normal_bf16(11, (t, nq, d))
    k = synth.normal_bf16(12, (prior + t, nkv, d))
    v = synth.normal_bf16(13, (prior + t, nkv, d))
    ref = T.op_causal_attention(q.astype(np.float64), k.astype(np.float64), v.astype(np.float64), prior)
    n_pages = (prior + t + 15) // 16
    pages = synth.page_permutation(14, n_pages + 5)[:n_pages]
    got = sts.op_attn_prefill(q, k, v, prior, pages, n_pages + 5)
    assert rel(got, ref) <= BF16_TOL
    # page order must not matter at all: same kernel, same tiles, only addresses differ
    got2 = sts.op_attn_prefill(q, k, v, prior, np.arange(n_pages, dtype=np.int32), n_pages + 5)
    assert np.array_equal(got, got2)


@pytest.mark.parametrize("nq,nkv,d,t,prior", [(4, 1, 128, 130, 5000), (2, 2, 64, 40, 3100), (8, 2, 128, 1, 4095), (2, 1, 128, 300, 6000), (1, 1, 64, 129, 17000)])
def test_prefill_attention_cuts_long_key_ranges(sts, nq, nkv, d, t, prior):
    """Few query tiles over many cached tokens: the key range is cut into parts whose outputs are merged (2 to 8 parts)."""
    q = synth.normal_bf16(81, (t, nq, d))
    k = synth.normal_bf16(82, (prior + t, nkv, d))
    v = synth.normal_bf16(83, (prior + t, nkv, d))
    np_ = (prior + t + 15) // 16
    pages = synth.page_permutation(84, np_ + 3)[:np_]
    got = sts.op_attn_prefill(q, k, v, prior, pages, np_ + 3)
    ref = T.op_causal_attention(q.astype(np.float64), k.astype(np.float64), v.astype(np.float64), prior)
    assert rel(got, ref) <= BF16_TOL


@pytest.mark.parametrize("nq,nkv,t,prior", [(512, 4, 1, 767), (512, 256, 31, 738), (256, 1, 200, 650), (512, 4, 65, 1000), (128, 4, 1500, 0), (128, 2, 250, 4099)])
@pytest.mark.parametrize("grow", [1.0, 8.0])
def test_prefill_attention_head_pairs(sts, nq, nkv, t, prior, grow):
    """Two heads of a group per workgroup. Key ranges that end at and around a tile's and a page's end, waves with fewer tiles than others,
    rows past the chunk, one group per pair and many, a range in parts; and (grow 8) scores that outgrow the first tile's maximum, with which
    the reference moves."""
    q = synth.normal_bf16(101, (t, nq, 128), grow)
    k = synth.normal_bf16(102, (prior + t, nkv, 128), grow)
    v = synth.normal_bf16(103, (prior + t, nkv, 128))
    if grow > 1:
        k[:64] *= 2.0 ** -6
    n_pages = (prior + t + 15) // 16
    pages = synth.page_permutation(104, n_pages + 2)[:n_pages]
    got, heads = sts.op_attn_prefill_form(q, k, v, prior, pages, n_pages + 2, heads=2)
    assert heads == 2 and np.isfinite(got).all()
    for h in (0, 1, nq // 2 - 1, nq - 2, nq - 1):
        g = h // (nq // nkv)
        ref = T.op_causal_attention(*(x.astype(np.float64) for x in (q[:, h:h + 1], k[:, g:g + 1], v[:, g:g + 1])), prior)
        assert rel(got[:, h:h + 1], ref) <= BF16_TOL, h


@pytest.mark.parametrize("nq,nkv,t,prior", [(512, 4, 1, 767), (512, 256, 31, 738), (256, 1, 200, 650), (4, 2, 65, 1000), (2, 1, 1500, 0), (8, 2, 250, 4099), (2, 1, 1, 0),
                                            (4, 1, 130, 63), (2, 1, 33, 95)])
@pytest.mark.parametrize("grow", [1.0, 1.7, 3.0, 8.0])
def test_prefill_attention_head_pairs_give_the_bits_of_one_head(sts, nq, nkv, t, prior, grow):
    """Both forms of the kernel multiply and add in the same order and move a row's reference maximum at the same scores (grow: never, in a few
    rows, in many, in all and repeatedly), so a layer's output does not depend on which of them a launch takes."""
    q = synth.normal_bf16(107, (t, nq, 128), grow)
    k, v = synth.normal_bf16(108, (prior + t, nkv, 128), grow), synth.normal_bf16(109, (prior + t, nkv, 128))
    if grow == 8.0:
        k *= np.float32(2.0) ** -(6 - np.minimum(6, np.arange(prior + t) // 90))[:, None, None]
    n_pages = (prior + t + 15) // 16
    pages = synth.page_permutation(110, n_pages + 2)[:n_pages]
    (one, h1), (two, h2) = (sts.op_attn_prefill_form(q, k, v, prior, pages, n_pages + 2, heads=h) for h in (1, 2))
    assert (h1, h2) == (1, 2)
    assert np.array_equal(one, two)
    taken = sts.op_attn_prefill_form(q, k, v, prior, pages, n_pages + 2)
    assert taken[1] == sts.attn_prefill_plan([t], [prior], nq, nkv, 128, 256)[2] and np.array_equal(taken[0], one)


@pytest.mark.parametrize("where", ["v_first", "v_late", "v_last", "k_first", "k_late", "k_minus", "q", "nan_v", "nan_k", "nan_q"])
@pytest.mark.parametrize("t,prior", [(130, 700), (250, 4099)])
def test_prefill_attention_head_pairs_with_infinities(sts, t, prior, where):
    """An infinity or a NaN in Q, K or V: the paired form multiplies probabilities of zero with values that the one-head form leaves out, so
    it hands such a workgroup to the one-head code. Same outputs as that, NaN for NaN; and rows that see none are finite."""
    nq, nkv, total = 4, 2, prior + t
    q = synth.normal_bf16(115, (t, nq, 128))
    k, v = synth.normal_bf16(116, (total, nkv, 128)), synth.normal_bf16(117, (total, nkv, 128))
    bad = np.nan if "nan" in where else -np.inf if where == "k_minus" else np.inf
    row = {"v_first": 3, "v_late": 601, "v_last": total - 1, "k_first": 70, "k_late": 601, "k_minus": 5, "nan_v": 601, "nan_k": 601}.get(where)
    x = {"v": v, "k": k, "q": q}[where.replace("nan_", "")[0]]
    x[t - 7 if x is q else row, 0, 11] = bad
    pages = synth.page_permutation(118, (total + 15) // 16)
    one, two = (sts.op_attn_prefill_form(q, k, v, prior, pages, len(pages), heads=h)[0] for h in (1, 2))
    assert np.array_equal(one, two, equal_nan=True)
    assert np.isfinite(two[:, 2:]).all() and not np.isfinite(two).all()      # the other KV group


@pytest.mark.parametrize("t,prior", [(1, 768), (31, 738), (200, 653), (65, 1001)])
def test_prefill_attention_head_pairs_ignore_what_lies_behind_the_context(sts, t, prior):
    """Keys and values that another sequence left behind the context, in the last page's free slots, with scores far above those of the
    context: the rows past the chunk must not see them, and no form's output depends on them."""
    nq, nkv, total = 4, 2, prior + t
    free = -total % 16
    assert free
    q = synth.normal_bf16(111, (t, nq, 128), 2.0)
    k, v = synth.normal_bf16(112, (total, nkv, 128), 2.0), synth.normal_bf16(113, (total, nkv, 128))
    k[:64] *= 2.0 ** -6
    left_k = np.broadcast_to(np.float32(64.0) * np.sign(q[-1, ::nq // nkv]), (free, nkv, 128))
    pages = synth.page_permutation(114, (total + 15) // 16)
    run = lambda heads, stale, kk, vv: sts.op_attn_prefill_form(q, kk, vv, prior, pages, len(pages), heads=heads, stale=stale)[0]
    want = run(1, 0, k, v)
    ks, vs = np.concatenate([k, left_k]), np.concatenate([v, np.full((free, nkv, 128), 2.0 ** 100, np.float32)])
    assert all((run(heads, free, ks, vs) == want).all() for heads in (1, 2))


def test_prefill_attention_head_pairs_near_the_end_of_fp32(sts):
    """Probabilities of up to 2^40 times values of 2^100: past fp32's range with the first tile's maximum as the reference, inside it where
    the reference moves."""
    nq, t, prior = 512, 2, 766
    q = np.full((t, nq, 128), 1.25, np.float32)
    k = np.zeros((prior + t, 1, 128), np.float32)
    k[200] = 2.0                                           # 320 / sqrt(128) log2(e) = 40.8
    v = synth.normal_bf16(106, (prior + t, 1, 128)) * np.float32(2.0 ** 100)
    got = sts.op_attn_prefill_form(q, k, v, prior, np.arange(48, dtype=np.int32), 48, heads=2)[0]
    ref = T.op_causal_attention(q[:, :1].astype(np.float64), k.astype(np.float64), v.astype(np.float64), prior)
    assert np.isfinite(got).all() and rel(got, np.broadcast_to(ref, got.shape)) <= BF16_TOL


@pytest.mark.parametrize("nq,nkv,d,ctx", [(8, 1, 128, [700, 257, 256, 17]), (8, 2, 128, [63, 65]), (4, 4, 64, [530, 513, 511, 33])])
def test_decode_attention_merges_many_chunks(sts, nq, nkv, d, ctx):
    """One page a chunk: 2 to 44 chunks a context, below, at and above what the merge kernel keeps in flight (16 or 32)."""
    q = synth.normal_bf16(65, (len(ctx), nq, d))
    k = synth.normal_bf16(66, (sum(ctx), nkv, d))
    v = synth.normal_bf16(67, (sum(ctx), nkv, d))
    got = sts.op_attn_decode(q, k, v, ctx, 1)
    off = 0
    for r, c in enumerate(ctx):
        kk, vv = k[off:off + c].astype(np.float64), v[off:off + c].astype(np.float64)
        for h in range(nq):
            ref = T.attend_one(q[r, h].astype(np.float64), kk[:, h // (nq // nkv)], vv[:, h // (nq // nkv)])
            assert rel(got[r, h], ref) <= BF16_TOL, (r, h)
        off += c


@pytest.mark.parametrize("nq,nkv,d,ctx,chunks", [(4, 4, 64, [32, 256, 1, 17, 100], 32), (4, 4, 64, [250, 33], 4),
                                                 (32, 8, 128, [1000, 40, 513, 16], 8), (8, 1, 128, [700], 5),
                                                 (32, 8, 128, [2048, 100], 16), (4, 4, 64, [129, 3], 1),
                                                 (32, 8, 128, [3000, 1025, 64], 64), (8, 1, 128, [1500], 33),
                                                 (16, 2, 128, [600, 31], 8), (4, 1, 64, [1100, 15], 64)])
def test_decode_attention(sts, nq, nkv, d, ctx, chunks):
    """`chunks` = pages per context chunk."""
    n = len(ctx)
    q = synth.normal_bf16(15, (n, nq, d))
    k = synth.normal_bf16(16, (sum(ctx), nkv, d))
    v = synth.normal_bf16(17, (sum(ctx), nkv, d))
    got = sts.op_attn_decode(q, k, v, ctx, chunks)
    off = 0
    for r, c in enumerate(ctx):
        kk, vv = k[off:off + c].astype(np.float64), v[off:off + c].astype(np.float64)
        for h in range(nq):
            ref = T.attend_one(q[r, h].astype(np.float64), kk[:, h // (nq // nkv)], vv[:, h // (nq // nkv)])
            assert rel(got[r, h], ref) <= BF16_TOL, (r, h)
        off += c


@pytest.mark.parametrize("nq,nkv,d,n_chunks", [(8, 1, 128, [2, 9, 16]), (8, 1, 128, [3, 17]), (8, 1, 128, [2, 9, 32, 33, 128]), (8, 2, 128, [65]), (4, 4, 64, [7, 16]),
                                               (4, 4, 64, [7, 17, 63, 64, 65, 128, 129]), (4, 1, 64, [5, 2])])
def test_decode_attention_adds_chunks_in_their_order(sts, nq, nkv, d, n_chunks):
    """The sums over a context's chunks (one page each) are taken in chunk order, whatever the number of chunks (16 and 17: two forms). Keys of zero make
    every probability 1 and every chunk's sum exact; element e has 2^24 in one chunk, -2^24 in a later one and small whole
    numbers elsewhere, so that fp32 sums in any other order come out different. The expected value is that fp32 sum, bit by bit."""
    ctx = [16 * c - 5 for c in n_chunks]
    rng = np.random.default_rng(91)
    q = synth.normal_bf16(92, (len(ctx), nq, d))
    k = np.zeros((sum(ctx), nkv, d), np.float32)
    v = np.zeros((sum(ctx), nkv, d), np.float32)
    want, off, other = np.empty((len(ctx), nq, d), np.float32), 0, 0
    for r, (c, n) in enumerate(zip(ctx, n_chunks)):
        part = rng.integers(1, 8, (n, nkv, d)).astype(np.float32)
        up = rng.integers(0, n - 1, (nkv, d))
        down = up + 1 + rng.integers(0, n, (nkv, d)) % (n - 1 - up)
        np.put_along_axis(part, up[None], np.float32(2.0 ** 24), 0)
        np.put_along_axis(part, down[None], np.float32(-2.0 ** 24), 0)
        v[off:off + 16 * n:16] = part                        # the first token of each page
        s = np.zeros((nkv, d), np.float32)
        for x in part:
            s = s + x
        want[r] = np.repeat(synth.to_bf16(s / np.float32(c)), nq // nkv, axis=0)
        other += int((s != part.sum(0, dtype=np.float64)).sum())
        off += c
    assert other > 0                                         # the order matters in these inputs
    assert np.array_equal(sts.op_attn_decode(q, k, v, ctx, 1), want)


def test_prefill_attention_with_no_room_for_more_parts(sts):
    """34 query tiles that would take 8 parts each, and room for 256: the first 32 are cut, the last two (16 and 17 thousand keys) are
    not. Rows of the first tile, of the last cut and the first uncut one, and the last row."""
    t, prior, d = 33 * 128 + 1, 16000, 64
    q = synth.normal_bf16(94, (t, 1, d))
    k = synth.normal_bf16(95, (prior + t, 1, d))
    v = synth.normal_bf16(96, (prior + t, 1, d))
    np_ = (prior + t + 15) // 16
    got = sts.op_attn_prefill(q, k, v, prior, synth.page_permutation(97, np_), np_)
    for a, b in ((0, 40), (31 * 128 + 100, 32 * 128 + 40), (t - 30, t)):
        ref = T.op_causal_attention(q[a:b].astype(np.float64), k[:prior + b].astype(np.float64), v[:prior + b].astype(np.float64), prior + a)
        assert rel(got[a:b], ref) <= BF16_TOL, (a, b)
