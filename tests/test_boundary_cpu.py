"""CPU-only checks of the C-ABI boundary: the library loads, exports every symbol the header
declares, its host packers emit exactly the oracle's bytes, and argument validation returns the
documented codes before anything touches a device."""
import ctypes
import os
import re

import numpy as np
import pytest

import paper_2410_21271_amd as eora
from paper_2410_21271_amd import binding
from tests.cases import QCase, SparseCase

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_library_exports_every_declared_symbol():
    text = open(os.path.join(ROOT, "include", "eora.h")).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    declared = set(re.findall(r"\b(eora_[a-z0-9_]+)\s*\(", text))
    assert declared, "no declarations found"
    assert declared == set(binding.EXPORTS)
    raw = ctypes.CDLL(eora.lib_path())
    for name in declared:
        assert getattr(raw, name) is not None


@pytest.mark.parametrize("w_bits,ab_bits,r", [(4, 16, 32), (3, 16, 64), (4, 4, 64), (3, 4, 128), (4, 16, 0), (2, 16, 32), (4, 3, 128)])
def test_host_packers_match_oracle_bytes(w_bits, ab_bits, r):
    QCase(100 + w_bits + r, 256, 48, 2, r, w_bits, 128, ab_bits, packer=eora)      # asserts inside
    QCase(200 + w_bits + r, 256, 32, 1, r, w_bits, 256, ab_bits, packer=eora)      # channel-wise group


def test_sparse_packer_matches_oracle_bytes():
    SparseCase(7, 256, 32, 1, 32, packer=eora)
    from tests.cases import SparseQCase
    SparseQCase(8, 512, 32, 1, 32, packer=eora)             # host packer = oracle layout, word for word
    SparseQCase(9, 512, 32, 1, 0, group=256, packer=eora)


def test_sizes():
    assert eora.qweight_bytes(4096, 4096, 4) == 4096 * 4096 // 2
    assert eora.qweight_bytes(4096, 4096, 3) == 4096 * 4096 * 3 // 8
    assert eora.qweight_bytes(4096, 4096, 2) == 4096 * 4096 // 4 and eora.qweight_bytes(4096, 4096, 1) == 0
    assert eora.qzeros_bytes(4096, 4096, 128) == 4096 * 32 // 2
    assert eora.qzeros_bytes(4096, 4096, 4096) == 4096 * 4          # channel-wise: one padded word per row
    assert eora.scales_bytes(4096, 4096, 128) == 4096 * 32 * 2
    assert eora.sp24_values_bytes(8192, 1024) == 8192 * 1024
    assert eora.sp24_indices_bytes(8192, 1024) == 8192 * 1024 // 8
    assert eora.sp24q4_tiles_bytes(8192, 1024) == 8192 * 1024 * 3 // 8 and eora.sp24q4_tiles_bytes(8192, 1000) == 0
    assert eora.sp24q4_meta_bytes(8192, 1024) == 1024 * 64 * 4
    assert eora.qweight_bytes(4096, 4100, 4) == 0 and eora.qweight_bytes(4096, 4096, 5) == 0
    assert eora.workspace_bytes(1, 4096, 4096, 128) >= 4 * 128
    assert eora.workspace_bytes(1, 4096, 4096, 1024) == 0


def test_packers_reject_bad_values():
    codes = np.zeros((16, 128), np.uint8)
    zeros = np.zeros((16, 1), np.uint8)
    scales = np.ones((16, 1), np.float16)
    codes[3, 5] = 8
    with pytest.raises(eora.EoraError) as ei:
        eora.pack_q(codes, zeros, scales, 3, 128)
    assert ei.value.status == -7
    eora.pack_q(codes, zeros, scales, 4, 128)
    zeros[0, 0] = 16
    with pytest.raises(eora.EoraError):
        eora.pack_q(codes, zeros, scales, 4, 128)
    with pytest.raises(eora.EoraError):
        eora.pack_sp24(np.zeros((16, 64), np.float16), np.zeros((16, 64), np.uint8))
    with pytest.raises(eora.EoraError):
        eora.pack_factor_f16(np.zeros((8, 32), np.float16))
    pos = np.tile(np.array([0, 1], np.uint8), (16, 32))
    c4 = np.zeros((16, 64), np.uint8)
    eora.pack_sp24q4(c4, pos, np.zeros((16, 1), np.uint8), np.ones((16, 1), np.float16), 128)
    c4[2, 7] = 16
    with pytest.raises(eora.EoraError) as ei:
        eora.pack_sp24q4(c4, pos, np.zeros((16, 1), np.uint8), np.ones((16, 1), np.float16), 128)
    assert ei.value.status == -7


def test_linear_q_validation_codes():
    """Every error path returns before a launch, so these calls are safe without a GPU: the
    pointers are never dereferenced."""
    L = eora.lib
    good = ctypes.c_void_p(0x1000)
    odd = ctypes.c_void_p(0x1008)
    null = ctypes.c_void_p(0)

    def call(x=good, qw=good, sc=good, qz=good, A=good, B=good, As=null, Bs=null, y=good, M=1, d_in=256, d_out=32,
             r=32, w_bits=4, group=128, ab_bits=16, ws=good, ws_bytes=1 << 24):
        return L.eora_linear_q(x, qw, sc, qz, A, B, As, Bs, y, M, d_in, d_out, r, w_bits, group, ab_bits, ws,
                               ws_bytes, null)

    assert call(x=null) == -1 and call(y=null) == -1 and call(A=null) == -1
    assert call(d_out=40) == -2 and call(d_in=200) == -2 and call(group=64) == -2 and call(group=384) == -2
    assert call(r=48) == -2 and call(r=1024) == -2 and call(M=-1) == -2
    assert call(w_bits=1) == -3 and call(w_bits=5) == -3 and call(ab_bits=8) == -3
    assert call(ab_bits=4, As=good, Bs=good, r=96) == -2 and call(ab_bits=4, r=64) == -1
    assert call(ab_bits=3, As=good, Bs=good, r=64) == -2 and call(ab_bits=3, r=128) == -1
    assert call(qw=odd) == -4 and call(y=odd) == -4 and call(ws=odd) == -4
    assert call(ws=null) == -5 and call(ws_bytes=16) == -5
    assert call(M=0) == 0                                   # empty input: nothing to do, nothing launched
    assert L.eora_linear_sp24(null, good, good, good, good, good, 1, 256, 32, 32, good, 1 << 24, null) == -1
    assert L.eora_linear_sp24(good, good, good, good, good, good, 1, 256, 32, 48, good, 1 << 24, null) == -2
    assert L.eora_linear_sp24(good, good, odd, good, good, good, 1, 256, 32, 32, good, 1 << 24, null) == -4
    assert L.eora_linear_sp24(good, good, good, good, good, good, 1, 256, 32, 32, good, 16, null) == -5
    # a group of layers that share x: validated member by member before anything is enqueued
    Q = eora.binding.QMember
    g, n0 = 0x1000, None

    def group(members, n=None, M=1, d_in=512, r=32, w_bits=4, group_=128, ab_bits=16, ws=good, ws_bytes=1 << 24, x=good):
        arr = (Q * max(1, len(members)))(*members)
        return L.eora_linear_q_group(x, arr, len(members) if n is None else n, M, d_in, r, w_bits, group_, ab_bits, ws,
                                     ws_bytes, null)

    ok = Q(g, g, g, g, g, n0, n0, g, 32)
    assert group([ok], n=0) == -2 and group([ok] * 5) == -2 and group([ok], x=null) == -1
    assert group([ok, Q(g, g, g, g, g, n0, n0, n0, 32)]) == -1            # second member without y
    assert group([ok, Q(g, g, g, g, g, n0, n0, g, 40)]) == -2             # d_out not a multiple of 16
    assert group([ok, Q(g, 0x1008, g, g, g, n0, n0, g, 32)]) == -4
    assert group([ok, ok], w_bits=5) == -3 and group([ok, ok], ws_bytes=16) == -5 and group([ok, ok], ws=null) == -5
    assert group([ok, ok], M=8, d_in=256, ws_bytes=16) == -5              # the member-by-member path validates too
    assert group([ok, ok], M=0) == 0
    assert L.eora_unpack_q(good, good, good, good, 256, 32, 5, 128, null) == -3
    assert L.eora_dequant_q(good, good, good, null, 256, 32, 4, 128, null) == -1
    assert L.eora_expand_sp24(good, odd, good, 256, 32, null) == -4
    sq = L.eora_linear_sp24q4
    assert sq(good, null, good, good, good, good, 1, 256, 32, 32, good, 1 << 24, null) == -1
    assert sq(good, good, good, good, good, good, 1, 200, 32, 32, good, 1 << 24, null) == -2
    assert sq(good, good, good, good, good, good, 1, 256, 32, 48, good, 1 << 24, null) == -2
    assert sq(good, odd, good, good, good, good, 1, 256, 32, 32, good, 1 << 24, null) == -4
    assert sq(good, good, good, good, good, good, 1, 256, 32, 32, good, 16, null) == -5
    assert sq(good, good, good, good, good, good, 0, 256, 32, 32, good, 1 << 24, null) == 0
    assert L.eora_expand_sp24q4(good, good, null, 256, 32, null) == -1
    assert L.eora_expand_sp24q4(good, good, good, 256, 40, null) == -2
    assert eora.status_string(-4) == "misaligned pointer"


def test_factors_validation_codes_and_sizes():
    """eora_factors validates before its first launch (no pointer is dereferenced on these paths)."""
    L = eora.lib
    good, odd, null = ctypes.c_void_p(0x1000), ctypes.c_void_p(0x1008), ctypes.c_void_p(0)

    def call(W=good, Wh=good, Xt=good, n=8, d_in=128, d_out=64, r=8, floor=1e-12, B=good, A=good, ws=good, ws_bytes=1 << 30):
        return L.eora_factors(W, Wh, Xt, n, d_in, d_out, r, floor, B, A, null, ws, ws_bytes, null, None)

    assert call(W=null) == -1 and call(Xt=null) == -1 and call(A=null) == -1
    assert call(d_in=127) == -2 and call(d_out=16386) == -2 and call(r=0) == -2 and call(r=65) == -2 and call(n=0) == -2
    assert call(floor=1.0) == -7 and call(floor=-1e-3) == -7 and call(floor=float("nan")) == -7
    assert call(ws=null) == -5 and call(ws_bytes=1 << 10) == -5 and call(ws=odd) == -4
    # five fp64 matrices (dW, G, V, dW', its copy) plus vectors and the r-row staging buffers
    n = eora.factors_workspace_bytes(4096, 4096, 128)
    assert 5 * 8 * 4096 * 4096 <= n <= 5 * 8 * 4096 * 4096 + (1 << 24)
    assert eora.factors_workspace_bytes(4096, 4097, 128) == 0 and eora.factors_workspace_bytes(64, 64, 65) == 0
    assert eora.status_string(-9) == "Jacobi sweeps did not converge"


def test_linear_q_multi_validation_codes():
    L = eora.lib
    good, odd, null = ctypes.c_void_p(0x1000), ctypes.c_void_p(0x1002), ctypes.c_void_p(0)

    def call(sel=good, A=good, M=4, r=32, n=2, w_bits=4, ab_bits=16, As=null, Bs=null, ws=good, ws_bytes=1 << 24):
        return L.eora_linear_q_multi(good, good, good, good, A, good, As, Bs, sel, good, M, 256, 32, r, n, w_bits, 128, ab_bits,
                                     ws, ws_bytes, null)

    assert call(sel=null) == -1 and call(A=null) == -1 and call(sel=odd) == -4
    assert call(n=0) == -2 and call(r=16) == -2 and call(r=0) == -2 and call(n=17) == -2
    assert call(ab_bits=4, r=64, As=good, Bs=good) == -2 and call(ab_bits=4, r=128, n=2) == -1
    assert call(w_bits=5) == -3 and call(ws=null) == -5 and call(ws_bytes=16) == -5
    assert call(M=0) == 0


def test_bench_refuses_more_than_one_gpu():
    """bench.py measures one GPU's share; asking for more ends with a message and a non-zero status
    before anything touches a GPU."""
    import os
    import subprocess
    import sys
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    p = subprocess.run([sys.executable, os.path.join(root, "bench.py"), "--gpus", "2"], capture_output=True, text=True, timeout=120)
    assert p.returncode != 0 and "not supported" in p.stderr and p.stdout.strip() == ""


def test_factors_store_f16_validation_codes():
    L = eora.lib
    good, odd, null = ctypes.c_void_p(0x1000), ctypes.c_void_p(0x1008), ctypes.c_void_p(0)

    def call(B=good, A=good, d_in=256, d_out=32, r=32, balance=1, At=good, Bt=good, scratch=good, nbytes=8 * 32):
        return L.eora_factors_store_f16(B, A, d_in, d_out, r, balance, At, Bt, scratch, nbytes, null)

    assert call(B=null) == -1 and call(At=null) == -1
    assert call(d_in=250) == -2 and call(d_out=24) == -2 and call(r=16) == -2 and call(r=0) == -2
    assert call(At=odd) == -4 and call(scratch=odd) == -4
    assert call(scratch=null) == -5 and call(nbytes=8 * 31) == -5


def test_factors_store_q_validation_codes():
    L = eora.lib
    good, odd, null = ctypes.c_void_p(0x1000), ctypes.c_void_p(0x1008), ctypes.c_void_p(0)

    def call(B=good, A=good, d_in=256, d_out=32, r=128, bits=4, balance=1, Aq=good, As=good, Bq=good, Bs=good, scratch=good,
             nbytes=8 * 128):
        return L.eora_factors_store_q(B, A, d_in, d_out, r, bits, balance, Aq, As, Bq, Bs, scratch, nbytes, null)

    assert call(B=null) == -1 and call(As=null) == -1 and call(bits=16) == -3 and call(bits=2) == -3
    assert call(d_in=192) == -2 and call(d_out=24) == -2 and call(r=96) == -2 and call(r=64, bits=3) == -2
    assert call(Bq=odd) == -4 and call(scratch=null) == -5 and call(nbytes=8) == -5


def test_linear_sp24_group_validation_codes():
    L = eora.lib
    S = eora.binding.SpMember
    g, null = 0x1000, ctypes.c_void_p(0)
    good = ctypes.c_void_p(g)

    def call(members, n=None, M=1, d_in=256, r=32, ws=good, ws_bytes=1 << 24, x=good):
        arr = (S * max(1, len(members)))(*members)
        return L.eora_linear_sp24_group(x, arr, len(members) if n is None else n, M, d_in, r, ws, ws_bytes, null)

    fp = S(g, g, None, None, g, g, g, 32)
    q4 = S(None, None, g, g, g, g, g, 32)
    # (only error paths and the empty batch are called: nothing here may reach a launch)
    assert call([fp], n=0) == -2 and call([fp] * 5) == -2 and call([fp], x=null) == -1
    assert call([fp, q4]) == -1                                   # members of different kinds
    assert call([fp, S(g, g, None, None, g, g, None, 32)]) == -1  # no y
    assert call([q4, S(None, None, g, g, g, g, g, 40)]) == -2
    assert call([fp, S(g, 0x1008, None, None, g, g, g, 32)]) == -4
    assert call([fp, fp], r=48) == -2 and call([fp, fp], ws=null) == -5 and call([fp, fp], ws_bytes=16) == -5
    assert call([fp, fp], M=0) == 0


@pytest.mark.parametrize("M,d_in,d_out,r", [(333, 4096, 4096, 128), (128, 4096, 16384, 0), (640, 14336, 4096, 256),
                                            (1024, 28672, 2048, 512), (1023, 28672, 1040, 128)])
def test_parts_of_a_prompt_never_need_more_than_their_room(M, d_in, d_out, r):
    """The fp32 outputs of the parts (4 * M * d_out bytes each) fit the room they are given to the byte, also where a
    room of one byte too few, as a float, is the room itself."""
    most = eora.debug_prefill_parts(M, d_in, d_out, r, 1 << 62)
    assert most > 1
    for parts in range(2, 9):
        need = parts * 4 * M * d_out
        for room in (need - 1, need - 16, need - 64, need, need + 1):
            got = eora.debug_prefill_parts(M, d_in, d_out, r, room)
            assert got == 1 or got * 4 * M * d_out <= room, (parts, room - need, got)
    assert eora.debug_prefill_parts(M, d_in, d_out, r, most * 4 * M * d_out) == most
    assert eora.debug_prefill_parts(M, d_in, d_out, r, 0) == 1


def _plan(M, d_in, d_outs, r):
    n = len(d_outs)
    ws = max([eora.workspace_bytes_group(M, d_in, r, n)] + [eora.workspace_bytes(M, d_in, d, r) for d in d_outs])
    return eora.debug_prefill_plan(M, d_in, d_outs, r, ws)


@pytest.mark.parametrize("M,d_in,d_outs,r,parts", [
    (1408, 1024, (656,), 0, 1), (175, 1024, (6976,), 256, 1), (276, 1152, (6880,), 128, 1), (189, 1152, (9392,), 128, 1),
    (336, 1280, (2432, 2720), 128, 1), (333, 14336, (4096,), 128, 8), (1014, 5120, (1680,), 128, 4), (2048, 14336, (4096,), 256, 2),
    (192, 1024, (816,), 256, 2), (199, 1024, (752,), 256, 2), (176, 1024, (560,), 128, 2), (378, 1280, (1008,), 128, 3)])
def test_short_contractions_of_a_prompt_stay_whole(M, d_in, d_outs, r, parts):
    """Parts of the main GEMM where both sides were timed on the GPU: cutting a short contraction costs more than it gives
    (16.5 us whole, 19.1 in two parts; 32.9 and 36.1; 34.2 and 38.1; 34.1 and 37.9; 35.3 and 38.6), a long one is cut, and a
    short one whose parts are a few hundred rows (32.0 us whole, 30.8 in two; 31.8 and 30.9; 29.3 and
    27.7; 32.3 in two and 31.3 in three)."""
    assert _plan(M, d_in, d_outs, r)[1] == parts


@pytest.mark.parametrize("M,d_in,d_outs,r,plan", [
    (512, 4096, (4096, 1024, 1024), 0, (128, 2, True)), (968, 3072, (688, 1040, 1424), 0, (128, 2, True)), (595, 2048, (5952,), 0, (128, 1, True)),
    (1024, 4096, (4096,), 0, (128, 2, True)), (1024, 28672, (8192,), 0, (128, 1, True)), (1044, 8064, (9600, 4432), 0, (128, 1, True)),
    (793, 3072, (8784, 5056, 3840), 0, (128, 1, True)), (2048, 1024, (4096,), 0, (128, 1, False)), (1024, 28672, (8192,), 128, (128, 1, False))])
def test_tiles_of_a_prompt_without_factors(M, d_in, d_outs, r, plan):
    """Tokens of a tile, parts and kernel of calls without factors where both sides were timed on the GPU: 128 tokens in fewer parts
    (41.5 us in larger tiles, 40.5; 35.7 and 33.9; 30.2 and 28.7), and from 32 steps on prefill128.hip at any number of workgroups
    (46.0 us on the other, 44.3; 453 and 432; 236.5 and 215.6; 106.3 and 94.1)."""
    tokens, parts, _, by128, _ = _plan(M, d_in, d_outs, r)
    assert (tokens, parts, by128) == plan


@pytest.mark.parametrize("M,d_in,d_outs,r,parts", [
    (1262, 1280, (1632, 1552), 256, 5), (1194, 1024, (752, 1296, 2832), 128, 8), (604, 1280, (1728, 1008, 2736), 256, 5),
    (1384, 1024, (1232, 1664, 2672), 256, 1), (1814, 1536, (656, 9216, 2512), 128, 3),
    (2028, 2688, (640, 560), 128, 7), (1207, 2304, (1328, 1648), 256, 6), (1179, 2048, (2288,), 256, 8), (823, 3072, (3040, 1984), 256, 8),
    (2048, 4096, (4096,), 256, 4), (2048, 14336, (4096,), 256, 8), (333, 14336, (4096,), 128, 38)])
def test_parts_of_a_prompts_down_projection(M, d_in, d_outs, r, parts):
    """Parts of t's contraction where both sides were timed on the GPU: a short one in as many as are one round of workgroups (40.3
    us a call instead of 45.2 in two; 36.0 instead of 39.0 whole; 41.0 instead of 43.3; up to 24 groups: 51.0 instead of 52.7, 54.4
    instead of 56.7, 47.3 instead of 48.2, 64.1 instead of 64.9), but not in more than a round (45.7 us
    whole, 52.1 in eight parts)."""
    assert _plan(M, d_in, d_outs, r)[2] == parts


@pytest.mark.parametrize("M,d_in,d_outs,r,shared", [
    (427, 2048, (752, 512), 256, False), (333, 14336, (4096,), 128, False), (715, 3072, (2144,), 256, False), (2048, 14336, (4096,), 256, True)])
def test_parts_of_a_prompt_lie_apart_where_there_is_room(M, d_in, d_outs, r, shared):
    """The main GEMM's parts behind t's in a workspace of the right size (34.8 us a call; in their place 37.7); in their place only
    where the room is not enough for both (2048 tokens: 16 + 64 MiB of 64)."""
    plan = _plan(M, d_in, d_outs, r)
    assert plan[1] > 1 and plan[2] > 1 and plan[4] == shared


@pytest.mark.parametrize("M,d_in,d_out", [(333, 1 << 20, 4096), (400, 8421376, 4096), (512, 8421504, 4096), (1000, 11 << 20, 8192), (2048, 1 << 24, 4096),
                                          (2048, 17 << 20, 4096), (512, 1 << 25, 4096), (2048, 1 << 27, 4096)])
def test_rows_of_x_in_a_tile_stay_within_32_bit_offsets(M, d_in, d_out):
    """The kernel with 32-bit offsets takes a tile only if its last row's last byte has one (and row times columns is a whole
    number of 31 bits); beyond, 128 tokens on the kernel that indexes with 64 bits."""
    tokens, _, _, by128, _ = eora.debug_prefill_plan(M, d_in, [d_out], 0, 1 << 62)
    assert by128 or ((tokens - 1) * d_in < 2 ** 31 and (tokens - 1) * d_in * 2 + 128 + 3072 < 2 ** 32), (tokens, by128)


@pytest.mark.parametrize("d_in,d_out", [(4096, 4096), (14336, 4096), (28672, 8192), (1152, 272)])
def test_workspace_sizes_never_shrink_with_tokens_or_rank(d_in, d_out):
    """A workspace of the size of the largest (M, r) serves smaller calls too, with everything they would have asked for
    themselves: the sizes never shrink as M, r or the number of members grows, and hold 12 MiB for partial outputs from
    five tokens and 48 MiB from 128 tokens on, beyond what the calls work with at least."""
    least = eora.workspace_bytes(1, 128, 16, 0)
    Ms = [1, 4, 5, 16, 64, 100, 127, 128, 129, 333, 1000, 1024, 1025, 2048, 2500, 4096, 4097, 4737, 5000, 8192, 9000, 20000, 40000, 100000]
    rs = [0, 32, 64, 96, 128, 160, 256, 320, 384, 512]
    sizes = [lambda M, r: eora.workspace_bytes(M, d_in, d_out, r)] + [
        lambda M, r, n=n: eora.workspace_bytes_group(M, d_in, r, n) for n in (1, 2, 3, 4)]
    for size in sizes:
        table = np.array([[size(M, r) for r in rs] for M in Ms], dtype=np.int64)
        assert (np.diff(table, axis=0) >= 0).all() and (np.diff(table, axis=1) >= 0).all()
        assert (table[2] - least >= 0).all()
    for a, b in zip(sizes[1:], sizes[2:]):
        assert all(a(M, r) <= b(M, r) for M in Ms for r in rs)
    for M in (5, 127, 128, 1024, 1025, 8192):
        room = (12 << 20) if M < 128 else (48 << 20)
        for size in sizes:
            assert size(M, 0) >= room
            assert size(M, 128) >= room + 2 * (M if M >= 128 else 0) * 128


def test_calibration_tokens_beyond_32_bit_offsets():
    """A tile of the Gram product spans 64 rows of n_tokens floats: 32-bit byte offsets are taken only as long as row 63's last
    byte has one."""
    assert eora.debug_factors_near(1) and eora.debug_factors_near(8192)
    for n in (17_043_000, 17_043_521, 17_043_522, 17_100_000, 2 ** 31 - 1):
        assert eora.debug_factors_near(n) == (4 * (63 * n + 31 + 1) <= 2 ** 32 - 1), n
    assert eora.debug_factors_near(17_043_000) and not eora.debug_factors_near(17_043_522)


def test_import_without_torchs_private_stream_functions():
    """Host packers and size queries need no GPU: they work with a torch that lacks the private functions behind the current
    stream, and the stream of a device call then comes from torch.cuda.current_stream()."""
    import subprocess
    import sys
    code = """
import types
import torch
for name in ("_cuda_getDevice", "_cuda_getCurrentRawStream"):
    if hasattr(torch._C, name):
        delattr(torch._C, name)
import numpy as np
import paper_2410_21271_amd as eora
from paper_2410_21271_amd import binding
assert eora.qweight_bytes(256, 32, 4) == 256 * 32 // 2
assert eora.pack_factor_f16(np.zeros((16, 32), dtype=np.float16)).size > 0
torch.cuda.current_stream = lambda: types.SimpleNamespace(cuda_stream=77)
torch.cuda.is_initialized = lambda: True
assert binding._stream() == 77
"""
    p = subprocess.run([sys.executable, "-c", code], capture_output=True, text=True, cwd=ROOT)
    assert p.returncode == 0, p.stderr[-2000:]


def test_parts_of_the_calibration_products_are_the_cheapest_that_fit():
    """Algorithm 1's products of 65 to 511 tiles: rounds of two workgroups a compute unit make the time rise and fall with the parts, so
    a number that the scratch does not hold must not be cut down to one that is dearer than another that fits.  Products of the subspace iteration at
    every multiple of 128 from 512 to 3072 (p vectors of length m, what its buffers leave of k x k doubles), and others."""
    def cost(c, tiles, M, N, K):
        left = tiles * c % 512
        column = 0.08 * (tiles * c // 512) + (0 if left == 0 else 0.052 if left <= 256 else 0.08)
        return column * K / c + (4 + 4e-6 * M * N * c if c > 1 else 0)

    def check(M, N, K, room):
        tiles, got = -(-M // 64) * -(-N // 64), eora.debug_factors_parts(M, N, K, room)
        most = max(1, min(K // 128, room // (M * N)))
        if K < 512 or tiles >= 512:
            assert got == 1
        elif tiles <= 64:
            assert got == min(256 // tiles, most)
        else:
            assert 1 <= got <= min(8, most)
            best = min(cost(c, tiles, M, N, K) for c in range(1, min(8, most) + 1))
            assert cost(got, tiles, M, N, K) <= best * (1 + 1e-5), (M, N, K, room, got)

    for m in range(512, 3073, 128):
        for r in range(32, 257, 32):
            p = (max(2 * r, r + 64) + 127) // 128 * 128
            if p <= m // 4:
                for k in (m, m + 128, 2 * m):
                    check(p, m, m, k * k - 2 * p * m - 3 * p * p)
                    check(p, k, m, k * k)
    for M, N, K, room in ((384, 2170, 2170, 10 ** 7), (64, 64, 512, 10 ** 6), (256, 4096, 4096, 0), (300, 5000, 511, 10 ** 8), (512, 4096, 640, 10 ** 8), (100, 100, 9000, 10 ** 6)):
        check(M, N, K, room)
    room = lambda p, m: m * m - 2 * p * m - 3 * p * p
    assert eora.debug_factors_parts(384, 2176, 2176, room(384, 2176)) == 2        # five are the cheapest of all; three, which fit, are dearer than two
    assert eora.debug_factors_parts(512, 3072, 3072, room(512, 3072)) == 2        # three fit
    assert eora.debug_factors_parts(512, 2560, 2560, room(512, 2560)) == 2        # no more fit
    assert eora.debug_factors_parts(0, 64, 512, 0) < 0
