"""Every GEMM kernel is run by some case here, and the case says by which: the rules that pick a kernel are host code, so
the CPU part of this file fails when a rule moves a case to another kernel and leaves one without a test.

Numbers (GPU part) against float64: tolerance 1e-2 of the largest value for bf16 results (one rounding is 2^-9 of a value),
1e-5 for fp32 ones (K products of the inputs, which are exact, summed in fp32 in some order)."""
import ctypes as C

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import transformer as ot          # noqa: E402
from paper_2410_07192_amd import synth        # noqa: E402

KERNELS = ("f32 fma", "bf16 generic", "ring 32x32", "ring 32x64", "ring 64x64", "ring 128x64", "tile 256x256",
           "tile 256x192", "tile 128x128", "tile 128x128 deep", "tile 256x128", "tile 128x64", "ring 32x32 deep",
           "ring 32x64 deep", "ring 64x64 deep", "tile 256x256 16")
EPI = {"plain": 0, "bias": 1, "gelu": 3, "resid": 5, "pre": 19, "dact": 8, "sum": 32}   # sum: fp32 result, accumulated


def route(dtype, M, N, K, epi="plain", misaligned=False):
    """Kernel and number of K slices of a product."""
    from paper_2410_07192_amd import binding as pf
    f = pf.lib.pf_gemm_route
    f.restype, f.argtypes = C.c_int32, [C.c_int32, C.c_int64, C.c_int64, C.c_int64, C.c_int32, C.c_int32]
    f32 = dtype == "f32"
    r = f(pf.PF_DTYPE_F32 if f32 else pf.PF_DTYPE_BF16, M, N, K, EPI[epi],
          int(misaligned) | (2 if f32 or epi == "sum" else 0))
    return KERNELS[r & 255], r >> 8


ALL = tuple(EPI)
# dtype, M, N, K, epilogues, kernel, K slices
PATHS = [
    # K no multiple of 64 on more tiles than the ring kernel takes: ragged, whole along M and N
    ("bf16", 1800, 2300, 200, ALL, "bf16 generic", 1),
    ("bf16", 2048, 1792, 72, ALL, "bf16 generic", 1),
    # fp32 rows that are not whole 16-byte chunks
    ("f32", 65, 99, 37, ALL, "f32 fma", 1),
    ("f32", 130, 70, 6, ALL, "f32 fma", 1),
    # fp32, large C and short K: aligned rows on the same kernel
    ("f32", 2047, 770, 16, ALL, "f32 fma", 1),
    # fp32 on every tile of the ring kernel
    ("f32", 97, 260, 36, ALL, "ring 32x32", 1),
    ("f32", 1000, 260, 36, ALL, "ring 32x64", 1),
    ("f32", 1023, 516, 36, ALL, "ring 64x64", 1),
    ("f32", 2047, 772, 64, ALL, "ring 128x64", 1),
    # and on its forms with two stages a wave: one to three steps a wave, the last one short or missing
    ("f32", 611, 516, 1060, ALL, "ring 32x32 deep", 1),
    ("f32", 2333, 516, 1796, ALL, "ring 32x32 deep", 1),
    ("f32", 611, 516, 268, ALL, "ring 32x64 deep", 1),
    ("f32", 1023, 1020, 260, ALL, "ring 64x64 deep", 1),
    ("f32", 1023, 1022, 1060, ALL, "ring 64x64 deep", 1),
    ("bf16", 7, 516, 1088, ALL, "ring 32x32 deep", 1),
    ("bf16", 333, 518, 1096, ALL, "ring 32x32 deep", 1),
    ("bf16", 333, 2044, 2312, ALL, "ring 64x64 deep", 1),
    # the tiled kernels: rows in 16- and 8-byte pieces and element by element, ragged along M, mostly along N
    ("bf16", 5000, 2368, 2048, ALL, "tile 256x256", 1),
    ("bf16", 5000, 2372, 2048, ("dact",), "tile 256x256", 1),
    ("bf16", 1999, 6156, 192, ("plain", "bias", "gelu", "resid", "pre", "sum"), "tile 256x256", 1),
    ("bf16", 5000, 2370, 2048, ("plain", "bias", "gelu", "resid", "pre", "sum"), "tile 256x256", 1),
    ("bf16", 5000, 2370, 4096, ("dact",), "tile 256x256", 1),
    ("bf16", 4000, 4088, 2112, ALL, "tile 256x256 16", 1),
    ("bf16", 4000, 4092, 2048, ALL, "tile 256x256 16", 1),
    ("bf16", 4000, 4090, 2048, ("plain", "bias", "gelu", "resid", "pre", "sum"), "tile 256x256 16", 1),
    ("bf16", 4001, 8184, 576, ("plain", "bias", "gelu", "resid", "pre", "sum"), "tile 256x256 16", 1),   # two rounds, nine steps
    ("bf16", 1300, 6152, 128, ALL, "tile 256x192", 1),
    ("bf16", 1300, 6156, 128, ALL, "tile 256x192", 1),
    ("bf16", 1300, 6154, 512, ALL, "tile 256x192", 1),
    ("bf16", 1659, 3072, 64, ALL, "tile 128x128", 1),
    ("bf16", 8292, 2370, 64, ALL, "tile 128x128", 1),
    ("bf16", 8292, 2372, 64, ("gelu", "pre", "dact"), "tile 128x128", 1),
    ("bf16", 3841, 1928, 3008, ("plain", "bias", "gelu", "resid", "pre", "dact"), "tile 256x128", 1),
    ("bf16", 1500, 776, 192, ("plain", "bias", "gelu", "resid", "dact"), "tile 128x64", 1),
    # K split over workgroups that have their CU to themselves (four LDS stages), ragged and whole, and that share it
    ("bf16", 100, 768, 16384, ("sum",), "tile 128x128 deep", 8),
    ("bf16", 1100, 512, 8192, ("sum",), "tile 128x128 deep", 4),
    ("bf16", 384, 3072, 4096, ("sum",), "tile 128x128 deep", 2),
    ("bf16", 900, 516, 16384, ("sum",), "tile 128x128", 8),
    ("bf16", 1024, 3072, 16384, ("sum",), "tile 128x128", 2),
]


@pytest.mark.parametrize("dtype,M,N,K,epis,kernel,splits", PATHS)
def test_the_case_runs_on_the_kernel_it_is_for(dtype, M, N, K, epis, kernel, splits):
    assert {route(dtype, M, N, K, e) for e in epis} == {(kernel, splits)}


def test_every_kernel_has_a_case():
    assert {p[5] for p in PATHS} == set(KERNELS)


# what other GPU tests are for: large tiles on one to five K steps with ragged edges, edge tiles, grids that do not fill the
# chip, rows in pieces
MOST = ("plain", "bias", "resid", "sum")
ROUNDED = ("gelu", "resid", "dact")


@pytest.mark.parametrize("M,N,K,epis,kernel", [
    (8292, 2368, 128, MOST, "tile 256x192"), (4196, 2372, 64, MOST + ("gelu", "pre"), "tile 256x192"),
    (4196, 3112, 64, MOST, "tile 256x256"), (8292, 3112, 128, MOST, "tile 256x256"),
    (8292, 3112, 192, MOST + ("gelu", "pre"), "tile 256x256"), (4196, 6152, 320, MOST + ("gelu", "pre"), "tile 256x256"),
    (8292, 3108, 64, MOST, "tile 256x256"), (1300, 6152, 128, ROUNDED, "tile 256x192"),
    (5000, 2368, 2048, ROUNDED, "tile 256x256"), (1999, 2040, 64, ROUNDED, "tile 128x128 deep"),
    (1659, 3072, 64, ROUNDED, "tile 128x128"), (1999, 2044, 64, ALL, "tile 128x128 deep"),
    (1999, 2040, 320, ALL, "tile 128x128 deep"), (33, 36, 72, ALL, "ring 32x32"), (128, 2300, 776, ALL, "ring 32x64"),
    (450, 2044, 1992, ALL, "ring 64x64"), (1659, 764, 3072, ("bias", "gelu", "resid", "pre", "dact"), "ring 128x64")])
def test_other_gpu_cases_run_on_the_kernel_they_are_for(M, N, K, epis, kernel):
    assert {route("bf16", M, N, K, e)[0] for e in epis} == {kernel}


# The faster kernel at sizes where two were timed on MI355X (times in us, the chosen one first): the rules follow them.  Where the
# kernels have changed since and a third one is faster now, it comes last, after "not chosen".
@pytest.mark.parametrize("dtype,M,N,K,epi,kernels", [
    # ring kernel, one LDS stage a wave or two
    ("f32", 1024, 1024, 256, "bias", "ring 64x64"),
    ("f32", 1024, 1024, 320, "bias", "ring 64x64 deep"),     # 13.0 / 13.5
    ("f32", 1024, 1024, 1024, "bias", "ring 64x64 deep"),    # 24.4 / 33.7
    ("f32", 614, 2440, 740, "bias", "ring 64x64 deep"),      # 37.5 / 44.6
    ("f32", 600, 512, 320, "bias", "ring 32x64 deep"),       # 7.6 / 8.0
    ("f32", 699, 684, 6756, "plain", "ring 32x32 deep"),     # 84 / 101
    ("f32", 2329, 544, 4624, "plain", "ring 32x32 deep"),    # 142 / 167
    ("f32", 4700, 144, 1304, "pre", "ring 32x32 deep"),      # 735 tiles: 33.9 / 39.0
    ("bf16", 3, 952, 4224, "gelu", "ring 32x32 deep"),       # 7.6 / 8.1
    ("bf16", 46, 896, 1688, "gelu", "ring 32x32 deep"),      # 5.8 / 6.1
    ("bf16", 333, 2048, 8192, "resid", "ring 64x64 deep"),   # 29.0 / 29.9
    # fp32: FMA kernel against the best ring tile
    ("f32", 4096, 2048, 64, "bias", "f32 fma"),        # 28.8 / 44.8
    ("f32", 8192, 1024, 128, "bias", "f32 fma"),       # 44 / 46
    ("f32", 2048, 2048, 64, "bias", "f32 fma"),        # 18.7 / 24.0
    ("f32", 2048, 576, 32, "bias", "f32 fma"),         # 9.7 / 128x64 12.1; not chosen: 32x32 9.3
    ("f32", 2048, 576, 64, "bias", "ring"),            # 12.1 / 12.8; not chosen: 32x32 10.9
    ("f32", 2048, 1024, 96, "bias", "ring"),           # 13.2 / 16.8
    ("f32", 2048, 576, 128, "bias", "ring 64x64"),     # 12.4; 128x64 16.2, fma 20.8; not chosen: 32x32 10.9
    ("f32", 2048, 2048, 192, "bias", "ring 128x64"),   # 32.5; 64x64 32.7, fma 38.0
    ("f32", 2048, 576, 512, "bias", "ring 32x32"),     # 22.5; 64x64 27.9
    ("f32", 4096, 2048, 256, "bias", "ring 64x64"),    # 63.6 / 75.0
    ("f32", 4004, 5119, 316, "bias", "f32 fma"),       # columns not in fours: 211 / 64x64 251
    ("f32", 2958, 418, 80, "gelu", "f32 fma"),         # 16.1 / 128x64 21.4; not chosen: 32x32 13.9
    ("f32", 512, 1024, 256, "gelu", "ring"),           # a layer of d 256 on 512 tokens
    ("f32", 512, 256, 1024, "resid", "ring"),
    # K no multiple of 64: generic kernel against the best ring tile
    ("bf16", 128, 24576, 200, "plain", "bf16 generic"),    # 10.7 / 14.3
    ("bf16", 2048, 1536, 1000, "plain", "bf16 generic"),   # 20.5 / 21.8
    ("bf16", 2048, 1536, 2008, "plain", "ring"),           # 31.7 / 38.6
    ("bf16", 2048, 1536, 328, "resid", "bf16 generic"),    # 17.2 / 128x64 20.5; not chosen: 64x64 15.9
    ("bf16", 2048, 1536, 600, "sum", "bf16 generic"),      # 21.1 / 32x32 23.3; not chosen: 64x64 19.0
    ("bf16", 2048, 1536, 1000, "sum", "ring"),             # 23.8 / 27.6
    ("bf16", 1024, 2048, 104, "plain", "bf16 generic"),    # 7.7 / 8.2
    ("bf16", 1024, 2048, 328, "plain", "ring"),            # 10.2 / 10.9
    ("bf16", 1024, 2048, 104, "sum", "ring"),              # 10.3 / 11.8
    ("bf16", 512, 512, 40, "plain", "ring"),               # 3.5 / 6.3
    ("bf16", 1000, 3072, 104, "plain", "ring"),            # ragged: 12.6 / 15.3
    ("bf16", 2048, 512, 600, "sum", "ring"),               # weight gradients of 600 tokens, d 512
    # few rows, weights from memory: 128x128 against 32x64 ring tiles
    ("bf16", 32, 19968, 4992, "gelu", "tile 128x128 deep"),  # 49.7 / 51.3
    ("bf16", 24, 18856, 5760, "pre", "tile 128x128 deep"),   # 55.8 / 56.9
    ("bf16", 24, 18856, 5760, "dact", "tile 128x128 deep"),  # 56.7 / 56.9
    ("bf16", 16, 17408, 4352, "dact", "ring 32x64"),         # 42.2 / 44.4
    # partial tiles along N for the chosen shape, none for the other
    ("bf16", 4096, 3456, 2048, "bias", "tile 256x256"),      # 52.8 / whole 128x128 tiles 58.3
    ("bf16", 8192, 1664, 2048, "bias", "tile 256x256"),      # 52.1 / whole 128x128 tiles 56.8
    ("bf16", 1659, 960, 768, "resid", "tile 128x64"),        # 8.2 / 128x128 deep 9.6, ring 12.5
    ("bf16", 522, 2848, 64, "plain", "tile 128x64"),         # 4.6 / 128x128 deep 5.0
    ("bf16", 1659, 768, 768, "resid", "tile 128x64"),        # 8.1 / 128x128 deep 9.4
    # the 256x256 tile by its own rate, and what the epilogues cost it
    ("bf16", 4096, 10048, 2048, "plain", "tile 256x256"),    # 146 / 256x192 187, 128x128 172
    ("bf16", 8192, 50304, 1024, "plain", "tile 256x256"),    # 743 / 256x192 920
    ("bf16", 50304, 1024, 8192, "sum", "tile 256x256"),      # 752 / 256x192 977
    ("bf16", 8192, 2304, 2048, "bias", "tile 256x192"),      # 87.0 / 256x256 90.0; not chosen: 128x128 82.0
    ("bf16", 8192, 1024, 1024, "resid", "tile 128x128"),
    ("bf16", 8192, 9648, 320, "dact", "tile 128x128"),       # 138 / 256x192 154, 256x256 217
    ("bf16", 4096, 9648, 320, "pre", "tile 128x128"),        # 55 / 256x256 71
    ("bf16", 8192, 5002, 768, "bias", "tile 128x128"),       # odd rows: 131 / 256x192 155, 256x256 195
    # weight gradients over long K: split or not, or few small tiles
    ("bf16", 1024, 3072, 8192, "sum", "tile 128x128"),       # two slices 71.5 / unsplit pairs 88.0; not chosen: deep, unsplit, 60.0
    ("bf16", 64, 64, 8192, "sum", "ring 32x32"),             # 11.8 / eight slices 11.7
    ("bf16", 1024, 3072, 4096, "sum", "tile 128x128 deep"),  # unsplit 31.0 / two slices 46.2
    ("bf16", 384, 3072, 4096, "sum", "tile 128x128 deep"),   # two slices 23.2 / four 32.2, unsplit 27.2; not chosen: 128x64 21.1
    ("bf16", 1024, 1024, 8192, "sum", "ring 64x64"),         # 32.2 / two slices 32.4, four 32.5
    ("bf16", 768, 1536, 8192, "sum", "tile 128x128"),        # four slices 43.8 / unsplit 46.9; not chosen: deep, two slices, 34.0
    ("bf16", 1536, 512, 8192, "sum", "ring 64x64"),          # 30.4 / two slices 30.6; not chosen: deep, four slices, 27.2
    ("bf16", 100, 132, 16384, "sum", "ring 32x32"),          # 21.7; not chosen: deep, eight slices, 17.8
])
def test_the_faster_kernel_is_chosen(dtype, M, N, K, epi, kernels):
    assert route(dtype, M, N, K, epi)[0].startswith(kernels)


def test_one_stage_a_wave_where_it_is_faster():
    assert {route(*p)[0] for p in (("f32", 1024, 1024, 256), ("bf16", 333, 2048, 2048))} == {"ring 64x64"}   # 8.8 / 9.9, 10.7 / 11.2
    assert {route(*p)[0] for p in (("f32", 512, 512, 4096), ("bf16", 128, 768, 3072), ("bf16", 9, 768, 3072))} == {"ring 32x32"}
    assert {route("f32", M, N, K)[0] for M, N, K in ((600, 512, 256), (600, 512, 352), (600, 512, 544))} == {"ring 32x64"}


def test_16x16x32_mfmas_on_a_full_chip_and_long_k_only():
    # us, the chosen form first; "in": of a pass of layers with this product
    assert {route("bf16", *p)[0] for p in ((4096, 4096, 2048),            # 56.7 / 58.3
                                           (8192, 2048, 8192),            # 191 / 202
                                           (3840, 4352, 1088),            # 255 tiles: in 523 / 545
                                           (16384, 4904, 1472),           # five full rounds: in 3095 / 3217
                                           (8192, 6192, 1536),            # 800 tiles, filled to 0.78: in 2097 / 2162
                                           (17920, 3384, 832),            # filled to 0.96: in 1652 / 1697
                                           (4096, 7168, 2112))} == {"tile 256x256 16"}       # 448 tiles: alone 111 / 108
    assert {route("bf16", *p)[0] for p in ((4096, 4096, 768),             # 27.4 / 27.8
                                           (15632, 7936, 320),            # 111 / 127
                                           (18560, 1792, 448),            # 511 tiles: in 638 / 640
                                           (9600, 2816, 704),             # 418 tiles: in 625 / 631
                                           (3332, 3840, 960),             # 210 tiles: in 609 / 615
                                           (964, 10112, 13696),           # 160 tiles: 243 / 284
                                           (408, 28032, 10048),           # 220 tiles
                                           (1400, 9216, 4160))} == {"tile 256x256"}          # 216 tiles: 93 / 97


def test_two_slices_where_they_are_faster():
    # than pairs of 128x128 tiles that keep their K (unsplit, with a CU each, the first three take 60, 60 and 55 us now, two slices
    # 71, 71 and 67: the estimate does not see it)
    assert [route("bf16", M, N, K, "sum")[1] for M, N, K in
            ((1024, 3072, 8192), (3072, 1024, 8192), (2048, 1536, 8192), (1024, 3072, 4096), (2048, 2048, 8192))] == [2, 2, 2, 1, 1]


# The k-major weight-gradient kernel (C += A^T B): slices of K, the fastest first where more than one was timed (us).
@pytest.mark.parametrize("M,N,K,slices", [(832, 1472, 1152, 2),      # 15.4; one 21.2, four 22.4
                                          (1280, 1280, 2048, 2),     # 23.7; one 31.2, four 30.3
                                          (512, 2560, 1536, 2),      # 18.3; one 25.6, four 24.5
                                          (2304, 768, 2048, 2),      # 23.7; one 29.8, four 31.1
                                          (2304, 768, 1024, 1),      # 16.5; two 17.7
                                          (1024, 1024, 8192, 4),     # 39; two 49, eight 48
                                          (512, 1792, 12032, 4),     # 44.6; eight 49.5, two 69.2
                                          (4096, 1024, 8192, 2),     # 85; one 95, four 102
                                          (2048, 2048, 4096, 1),     # 55; two 58
                                          (4096, 1024, 1024, 1),     # 22.6; two 34.5
                                          (4608, 64, 256, 1),        # 8.7; two 9.6
                                          (64, 64, 704, 4),          # 8.1; two 9.3
                                          (64, 376, 256, 2),         # 7.5; one 8.3
                                          (50304, 1024, 8192, 1)])
def test_the_fastest_number_of_slices(M, N, K, slices):
    from paper_2410_07192_amd import binding as pf
    f = pf.lib.pf_gemm_tn_slices
    f.restype, f.argtypes = C.c_int32, [C.c_int64, C.c_int64, C.c_int64]
    assert f(M, N, K) == slices


def test_misaligned_operands_go_to_the_kernels_without_16_byte_copies():
    assert route("bf16", 128, 768, 768, misaligned=True) == ("bf16 generic", 1)
    assert route("f32", 128, 768, 768, misaligned=True) == ("f32 fma", 1)


def _product(dtype, M, N, K, epis):
    from paper_2410_07192_amd import binding as pf
    from paper_2410_07192_amd import device as dev
    md = pf.pf_model_desc()
    md.dtype = pf.PF_DTYPE_BF16 if dtype == "bf16" else pf.PF_DTYPE_F32
    rng = np.random.default_rng(M + N + K)

    def draw(shape, scale):
        a = (rng.standard_normal(shape) * scale).astype(np.float32)
        return synth.round_to_bf16(a) if dtype == "bf16" else a

    X, W, bias, R = draw((M, K), 1.0), draw((N, K), 0.05), draw((N,), 1.0), draw((M, N), 1.5)
    dX, dW, db, dR = (dev.storage_tensor(a, md) for a in (X, W, bias, R))
    p = X.astype(np.float64) @ W.astype(np.float64).T
    u = p + bias
    pre = dev.empty_storage((M, N), md)
    calls = {"plain": ({}, p), "bias": (dict(bias=db.data_ptr()), u),
             "gelu": (dict(bias=db.data_ptr(), gelu=1), ot.gelu(u)),
             "resid": (dict(bias=db.data_ptr(), resid=dR.data_ptr()), u + R),
             "pre": (dict(bias=db.data_ptr(), gelu=1, preact_out=pre.data_ptr()), ot.gelu(u)),
             "dact": (dict(dact_in=dR.data_ptr()), p * ot.gelu_grad(R.astype(np.float64)))}
    err = lambda got, ref: float(np.abs(got - ref).max() / np.abs(ref).max())
    tol = 1e-2 if dtype == "bf16" else 1e-5
    for e in epis:
        if e == "sum":
            before = rng.standard_normal((M + 1, N)).astype(np.float32)
            acc = torch.from_numpy(before).cuda()
            for _ in range(2):
                pf.pf_op_gemm(md.dtype, dX.data_ptr(), dW.data_ptr(), acc.data_ptr(), M, N, K, out_f32=1, accumulate=1)
            torch.cuda.synchronize()
            got = acc.cpu().numpy()
            assert err(got[:M], before[:M] + 2 * p) < 1e-5 and np.array_equal(got[M], before[M])
            continue
        out = dev.empty_storage((M + 1, N), md)          # one extra row behind C: must stay untouched
        out.zero_()
        pf.pf_op_gemm(md.dtype, dX.data_ptr(), dW.data_ptr(), out.data_ptr(), M, N, K, **calls[e][0])
        torch.cuda.synchronize()
        got = dev.read_storage(out, md)
        assert err(got[:M], calls[e][1]) < tol and not got[M].any(), e
        if e == "pre":
            assert err(dev.read_storage(pre, md), u) < tol


# Sums into an fp32 C of 96 M elements or more go past the caches (on tiled kernels with rows in pieces of 16 bytes).
LARGE_SUMS = [(10250, 9828, 64), (7162, 16380, 2048)]


@pytest.mark.parametrize("M,N,K,kernel", [a + (k,) for a, k in zip(LARGE_SUMS, ("tile 256x256", "tile 256x256 16"))])
def test_large_sums_run_on_tiled_kernels(M, N, K, kernel):
    assert M * N >= 96 << 20 and N % 4 == 0 and M % 256 and N % 256 and route("bf16", M, N, K, "sum") == (kernel, 1)


@pytest.mark.gpu
@pytest.mark.parametrize("M,N,K", LARGE_SUMS)
def test_numbers_of_large_sums(M, N, K):
    from paper_2410_07192_amd import binding as pf
    gen = torch.Generator(device="cuda")
    gen.manual_seed(M + N)
    X = torch.randn(M, K, device="cuda", generator=gen).to(torch.bfloat16)
    W = (torch.randn(N, K, device="cuda", generator=gen) * 0.05).to(torch.bfloat16)
    acc = torch.randn(M + 1, N, device="cuda", generator=gen)          # a row behind C: must stay untouched
    ref, last = acc[:M].double(), acc[M].clone()
    for _ in range(2):
        pf.pf_op_gemm(pf.PF_DTYPE_BF16, X.data_ptr(), W.data_ptr(), acc.data_ptr(), M, N, K, out_f32=1, accumulate=1)
    torch.cuda.synchronize()
    ref += 2 * (X.double() @ W.double().t())
    assert float((acc[:M] - ref).abs().max() / ref.abs().max()) < 1e-5 and torch.equal(acc[M], last)


# fp32 attention, heads in all, tokens, d_head: tiles or one thread per query (us, the chosen one first)
ATTENTION = [(4096, 16, 32, False),    # 27 / 68
             (1024, 8, 64, False),     # 17.6 / 25.6
             (2048, 24, 64, False),    # 47 / 53
             (2048, 48, 64, False),    # 92 / 111
             (2048, 4, 128, False),    # 55 / 78
             (2048, 32, 64, True),     # 47 / 60
             (2048, 64, 64, True),     # 96 / 125
             (2048, 16, 128, True),    # 86 / 139
             (512, 16, 32, True),      # 10.1 / 13.3
             (16, 1, 32, True),        # 6.0 / 6.9
             (16, 128, 64, True)]      # four sequences of 128 tokens, d 256: 7.7 / 129


@pytest.mark.parametrize("units,S,dh,tiles", ATTENTION)
def test_the_faster_fp32_attention_is_chosen(units, S, dh, tiles):
    from paper_2410_07192_amd import binding as pf
    f = pf.lib.pf_attention_f32_tiles
    f.restype, f.argtypes = C.c_int32, [C.c_int64, C.c_int64, C.c_int64, C.c_int32]
    assert {bool(f(units // h, S, h, dh)) for h in (1, 4, 16)} == {tiles}


@pytest.mark.gpu
@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("units,S,dh", [a[:3] for a in ATTENTION if not a[3]])
def test_numbers_of_many_short_fp32_sequences(units, S, dh, causal):
    from paper_2410_07192_amd import binding as pf
    from paper_2410_07192_amd import device as dev
    md = pf.pf_model_desc()
    md.dtype = pf.PF_DTYPE_F32
    h = 8
    B, d = units // h, h * dh
    rng = np.random.default_rng(S + dh)
    qkv = rng.standard_normal((B, S, 3 * d), dtype=np.float32)
    dq, out = dev.storage_tensor(qkv, md), dev.empty_storage((B, S, d), md)
    lse = torch.empty((B, h, S), dtype=torch.float32, device="cuda")
    pf.pf_op_attention(md.dtype, dq.data_ptr(), out.data_ptr(), B, S, h, dh, causal, lse.data_ptr())
    torch.cuda.synchronize()
    q, k, v = (ot.split_heads(qkv[..., i * d:(i + 1) * d].astype(np.float64), h) for i in range(3))
    ref = ot.merge_heads(ot.attention_probs(q, k, causal) @ v)
    s = q @ k.transpose(0, 1, 3, 2) / np.sqrt(dh)
    if causal:
        s = np.where(np.triu(np.ones((S, S), dtype=bool), 1), -np.inf, s)
    ref_lse = np.log(np.exp(s).sum(-1))
    assert np.abs(dev.read_storage(out, md) - ref).max() < 1e-5 * np.abs(ref).max()
    assert np.abs(lse.cpu().numpy() - ref_lse).max() < 1e-4


@pytest.mark.gpu
@pytest.mark.parametrize("dtype,M,N,K,epis,kernel,splits", PATHS)
def test_numbers_of_every_path(dtype, M, N, K, epis, kernel, splits):
    _product(dtype, M, N, K, epis)
