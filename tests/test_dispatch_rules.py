"""Which tiles a launch of the grouped bf16 GEMM takes: the rules are constant expressions, evaluated by the compiler on the host side alone (no GPU)."""
import os
import subprocess

import pytest

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2506_05229_amd", "csrc")
pytestmark = pytest.mark.skipif(not os.path.exists(HIPCC), reason="needs hipcc")


def holds(tmp_path, *facts):
    """Compiles `facts`, C++ conditions, as static assertions behind the dispatch's source; what fails is in the message."""
    source = tmp_path / "facts.hip"
    source.write_text('#include "gemm_mfma.h"\nusing namespace armt;\n'
                      "constexpr GemmShape product(int M, int N, int K) {\n"
                      "  GemmShape s{};\n"
                      "  s.M = M; s.N = N; s.K = K; s.lda = s.ldb = K; s.ldc = N; s.n0 = N;\n"
                      "  return s;\n}\n"
                      "constexpr GemmShape without_strip(int M) {\n"
                      "  GemmShape s = product(M, 2048, 2048);\n"
                      "  s.dbg = 32; s.a_rows = (M + 255) / 256 * 256;\n"
                      "  return s;\n}\n"
                      "constexpr GemmShape qkv(int M, int ldc2) {\n"
                      "  GemmShape s = product(M, 3072, 2048);\n"
                      "  s.n0 = 2048; s.n1 = 512; s.ldr = 64; s.ldc2 = ldc2; s.a_rows = (M + 255) / 256 * 256;\n"
                      "  return s;\n}\n" + "".join(f'static_assert({f}, "");\n' for f in facts))
    done = subprocess.run([HIPCC, "-std=c++17", "--offload-arch=gfx950", "--cuda-host-only", "-fsyntax-only", "-I", CSRC, str(source)],
                          capture_output=True, text=True)
    assert done.returncode == 0, done.stderr


def test_partial_round(tmp_path):
    """Up to half a round of 256 x 256 tiles behind whole ones runs as 128 x 128 tiles, whatever kernel the whole ones take."""
    cut = "mfma_round_cut<EPI_STORE_ACT>"
    holds(tmp_path,
          f"{cut}(product(272, 3072, 2048), 32, -1) == 256",      # 384 tiles, a strip behind a single M-tile: units of one tile
          f"{cut}(product(1040, 3072, 128), 12, -1) == 128",      # 576 tiles, two k-tiles: units of four
          f"{cut}(product(4352, 4352, 192), 1, -1) == 44",        # 289 tiles, M-groups of 6, 6 and 5 M-tiles: seven panels of the last one are cut off
          f"{cut}(product(4352, 4352, 128), 1, -1) == 44",
          f"{cut}(product(1040, 2048, 2048), 8, -1) == 0",        # one round
          f"{cut}(product(1040, 2048, 2048), 14, -1) == 0",       # 448 tiles: more than half a round is left
          f"{cut}(product(4352, 4352, 192), 1, 5) == 0")          # tiles asked for


def test_small_or_big_tiles(tmp_path):
    """128 x 128 tiles (6) as long as they fit the chip in one round, also where ragged edges make more than a quarter as many of 256 x 256."""
    pick = lambda g, *dims: f"mfma_pick_config(product({', '.join(map(str, dims))}), {g}, -1)"
    holds(tmp_path,
          f"{pick(4, 1040, 2048, 2048)} == 6 && {pick(11, 1040, 768, 768)} == 5",      # 512, 528
          f"{pick(3, 1100, 2300, 2048)} == 6 && {pick(5, 2100, 768, 768)} == 6",       # 486 and 510: 135 tiles of 256 x 256
          f"{pick(13, 500, 1280, 1024)} == 5")


def test_persistent_tile(tmp_path):
    """Rows that end in a strip of 16 take the persistent 256 x 256 tile also where one M-tile is all that the strip has in front of it, and so do products of
    one or two k-tiles, fewer than its copies are ahead."""
    holds(tmp_path,
          "tile256_shape<EPI_SWIGLU>(product(272, 8192, 2048))",
          "tile256_shape<EPI_STORE_ACT>(product(57 * 256 + 16, 2048, 2048))",      # M-groups of eight, the last of one
          "tile256_shape<EPI_STORE_ACT>(product(1040, 2048, 192))",
          "tile256_shape<EPI_RESID_F32>(product(1040, 2048, 128))",
          "tile256_shape<EPI_RESID_F32>(product(46080, 768, 64))",
          "tile256_short(product(1040, 2048, 128)) && !tile256_short(product(1040, 2048, 192))",
          "!tile256_shape<EPI_STORE_ACT>(product(1040, 2048, 0))")


def test_transposed_v(tmp_path):
    """The persistent tile stores V^T eight rows at a time, looking at the first: rows that are no multiple of eight stay with the tiles that look at each."""
    tile = "tile256_shape<EPI_QKV_ROPE>"
    holds(tmp_path, "mfma_regular_shape<256, 256, EPI_QKV_ROPE>(qkv(1036, 1152))", f"!{tile}(qkv(1036, 1152))", f"!{tile}(qkv(1047, 1152))",
          f"{tile}(qkv(1048, 1152))", f"{tile}(qkv(1040, 1152))", f"{tile}(qkv(1036, 0))")


def test_cut_without_strip(tmp_path):
    """Memory rows in an M-tile of their own (a switch of the tile configuration): the units of a cut launch still hold every tile."""
    facts = []
    for rows in (272, 1040, 2064, 2320, 14608):
        tiles = (rows + 255) // 256
        facts += [f"mfma_m_tiles(without_strip({rows})) == {tiles}",
                  f"mfma_unit_tile(mfma_units(without_strip({rows}), 9, 8), {tiles}, mfma_m_group(without_strip({rows})), 8, 1) == {9 * tiles * 8}",
                  f"mfma_m_tiles(product({rows}, 2048, 2048)) == {tiles - 1}"]
    holds(tmp_path, "mfma_round_cut<EPI_RESID_F32>(without_strip(1040), 15, -1) > 0", *facts)


def test_cut_inside_m_group(tmp_path):
    """The launches that tests on the device mean to cut inside an M-group: units per M-group are the panels."""
    residual = "mfma_round_cut<EPI_RESID_F32>(product(2320, 1280, 1024), 6, -1)"
    holds(tmp_path, f"{residual} == 56 && {residual} % 5 != 0",
          "mfma_round_cut<EPI_STORE_F32>(product(4352, 4096, 4352), 1, -1) % 16 != 0", "mfma_round_cut<EPI_RESID_F32>(product(4352, 4096, 4352), 1, -1) % 16 != 0")
