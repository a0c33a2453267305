"""CPU-only checks of the native library: it loads, exports every entry point the
header declares, validates arguments, plans launches, and its host packer writes
the specified layout (pinned against hand-derived bytes and the oracle's reader)."""
import json
import os
import re
import subprocess
import sys

import numpy as np
import pytest

import oracle
import paper_2509_18344_amd as ss
from paper_2509_18344_amd import _binding

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_library_exports_every_declared_symbol():
    lib = ss.load_library()
    header = open(os.path.join(ROOT, "include", "subspec.h")).read()
    names = set(re.findall(r"\b(subspec_[a-z_0-9]+)\s*\(", header))
    assert len(names) >= 9
    for n in names:
        assert hasattr(lib, n), n


def test_qpack_bytes():
    assert ss.subspec_qpack_bytes(4, 512, 256) == 512 * 256 // 2
    assert ss.subspec_qpack_bytes(3, 16, 128) == 768
    assert ss.subspec_qpack_bytes(2, 32, 256) == 2048
    assert ss.subspec_qpack_bytes(5, 16, 128) == 0
    assert ss.subspec_qpack_bytes(4, 8, 128) == 0
    assert ss.subspec_qpack_bytes(4, 16, 100) == 0


def _golden_rows(golden_dir):
    rows = []
    with open(os.path.join(golden_dir, "unpack_bytes.txt")) as f:
        for ln in f:
            if ln.strip() and not ln.startswith("#"):
                rows.append(ln.split())
    return rows


def test_host_packer_matches_golden_bytes(golden_dir):
    rows = _golden_rows(golden_dir)
    for bits in (2, 3, 4):
        codes = np.zeros((16, 128), np.uint8)
        expect = np.zeros(256 * bits, np.uint8)
        for b, n, k, q, off, val in rows:
            if int(b) != bits:
                continue
            codes[int(n), int(k)] = int(q)
            expect[int(off)] |= int(val, 16)
        out = np.zeros(256 * bits, np.uint8)
        ss.subspec_qpack_host(codes, bits, 16, 128, out)
        assert np.array_equal(out, expect), bits


@pytest.mark.parametrize("bits", [2, 3, 4])
def test_host_packer_round_trip_exhaustive(bits):
    # every code value at every position of a tile, plus a random multi-tile matrix
    N, K = 16, 128
    for v in range(2 ** bits):
        codes = np.full((N, K), v, np.uint8)
        out = np.zeros(N * K * bits // 8, np.uint8)
        ss.subspec_qpack_host(codes, bits, N, K, out)
        assert np.array_equal(oracle.unpack(out, bits, N, K), codes)
    rng = np.random.default_rng(bits)
    for N, K in [(16, 128), (48, 384), (32, 1024)]:
        codes = rng.integers(0, 2 ** bits, (N, K)).astype(np.uint8)
        out = np.zeros(N * K * bits // 8, np.uint8)
        ss.subspec_qpack_host(codes, bits, N, K, out)
        assert np.array_equal(oracle.unpack(out, bits, N, K), codes)


@pytest.mark.parametrize("M,N,K,bits,group,path,err", [
    (1, 512, 256, 5, 64, 0, "EUNSUPPORTED"),
    (1, 512, 256, 4, 32, 0, "EUNSUPPORTED"),
    (1, 512, 200, 4, 64, 0, "EUNSUPPORTED"),
    (1, 520, 256, 4, 64, 0, "EUNSUPPORTED"),
    (0, 512, 256, 4, 64, 0, "EUNSUPPORTED"),
    (129, 512, 256, 4, 64, 0, "EUNSUPPORTED"),
    (9, 512, 256, 4, 64, 1, "EUNSUPPORTED"),
    (4, 512, 256, 4, 64, 7, "EINVAL"),
    (4, -16, 256, 4, 64, 0, "EINVAL"),
    (4, 1 << 20, 1 << 13, 4, 64, 0, "EUNSUPPORTED"),   # N*K > 2^32
    (4, 16, (1 << 24) + 128, 4, 64, 0, "EUNSUPPORTED"),  # K > 2^24
])
def test_plan_rejects_bad_shapes(M, N, K, bits, group, path, err):
    with pytest.raises(ss.SubspecError) as ei:
        ss.subspec_qlinear_plan(M, N, K, bits, group, path)
    assert err in str(ei.value)


def test_plan_choices_are_consistent():
    for M in (1, 2, 3, 4, 5, 8, 9, 16, 17, 32, 33, 64, 65, 100, 128):
        for (N, K) in [(512, 256), (18944, 3584), (3584, 18944), (55296, 5120), (5120, 27648), (7168, 5120)]:
            for bits, group in [(4, 128), (3, 128), (2, 64), (4, 64)]:
                p = ss.subspec_qlinear_plan(M, N, K, bits, group)
                rb = p["row_blocks"]
                # row blocks: two of 16x16x32 tiles or any number of 32-row 32x32 tiles,
                # each block holding at least one row
                assert rb == 1 or (p["full_groups"] == 0 and (
                    (rb == 2 and p["mfma_rows"] == 16) or (p["mfma_rows"] == 32 and p["rows"] == 32))), p
                assert p["rows"] * rb >= M > p["rows"] * (rb - 1)
                KB = K // 128
                assert p["splits"] >= 1 and p["blocks_per_split"] % p["chunk_blocks"] == 0
                assert (p["splits"] - 1) * p["blocks_per_split"] < KB <= p["splits"] * p["blocks_per_split"]
                # teams split a workgroup's k-blocks (two on 32x32 tiles; every wavefront
                # of a small-batch launch); a layout mismatch between the binding and the
                # C struct would show here
                small = p["mfma_rows"] == 16 and p["teams"] > 1
                assert p["teams"] == 1 or (p["teams"] == 2 and p["mfma_rows"] == 32 and p["waves"] == 8) or (
                    small and M <= 16 and p["teams"] == p["waves"] and p["splits"] == 1 and p["rows"] in (4, 8, 16)), p
                cols = p["waves"] // p["teams"] * p["tiles_per_wave"] * 16
                assert p["col_groups"] == -(-N // cols)
                fg = p["full_groups"]
                assert 0 <= fg < p["col_groups"]
                grid = fg + (p["col_groups"] - fg) * p["splits"]
                assert p["grid"] == (-(-grid // 8) * 8 if small else grid)
                if fg:
                    # whole groups on a multiple of the CUs; the rest split at most
                    # once per CU
                    assert p["splits"] > 1 and fg % 256 == 0
                    assert (p["col_groups"] - fg) * p["splits"] <= 256
                # completion counters (16384 x 4 bytes), the per-group sums of x the
                # 32x32 kernel reads on taller tiles (fp32 [K/group][M], 256-byte
                # aligned), then the splits' fp32 partial sums: nothing the launch does
                # not read
                xs = -(-M * (K // group) * 4 // 256) * 256 if p["mfma_rows"] == 32 and p["rows"] > 64 else 0
                part_rows = rb * p["rows"] if rb > 1 else M
                partials = p["splits"] * part_rows * N * 4 if p["splits"] > 1 else 0
                expect = 65536 + xs + partials if (xs or partials) else 0
                assert p["workspace_bytes"] == expect, (M, N, K, bits, group, p)
    # 592 column groups on 256 CUs: 512 whole, the last 80 split three ways
    p = ss.subspec_qlinear_plan(1, 37888, 3584, 4, 128)
    assert (p["col_groups"], p["full_groups"], p["splits"], p["grid"]) == (592, 512, 3, 752)
    # automatic plan: GEMV only for one row of the larger weights (measured crossover),
    # MFMA from M = 2; small weights on matrix cores from one row on, without workspace
    assert ss.subspec_qlinear_plan(1, 37888, 3584, 4, 128)["path"] == ss.SUBSPEC_PATH_GEMV
    assert ss.subspec_qlinear_plan(2, 37888, 3584, 4, 128)["path"] == ss.SUBSPEC_PATH_MFMA
    for M in (1, 2, 8):
        p = ss.subspec_qlinear_plan(M, 512, 256, 4, 64)
        assert (p["path"], p["mfma_rows"], p["teams"], p["workspace_bytes"]) == (ss.SUBSPEC_PATH_MFMA, 16, 4, 0)
    # the small-batch lines: blocks a wavefront takes in a row, workgroups per CU
    for M, N, K, small in [(2, 3584, 20480, True), (2, 3584, 20608, False), (3, 512, 20480, True), (4, 512, 18432, True),
                           (4, 512, 18560, False), (4, 528, 20480, True), (4, 112, 18432, True),
                           (4, 112, 18560, False), (4, 128, 20480, True),
                           (4, 1024, 20480, True), (6, 2880, 14336, True), (7, 768, 13824, True), (7, 768, 13952, False),
                           (7, 464, 14336, True), (7, 176, 9216, False), (7, 192, 9216, True), (8, 2880, 12288, True),
                           (8, 2880, 13312, True), (8, 2880, 13440, False), (8, 464, 13824, True), (8, 464, 14208, False),
                           (8, 256, 9088, False), (8, 256, 9216, True), (8, 240, 9216, False), (8, 320, 9088, True),
                           (9, 9008, 1536, True), (10, 9008, 1536, False), (16, 8192, 1536, True),
                           (16, 8208, 1536, False)]:
        assert (ss.subspec_qlinear_plan(M, N, K, 4, 128)["teams"] > 1) == small, (M, N, K)
    p = ss.subspec_qlinear_plan(6, 4608, 3584, 4, 128)
    assert (p["mfma_rows"], p["rows"], p["tiles_per_wave"], p["teams"], p["grid"]) == (16, 8, 2, 16, 144)
    # launches that need no scratch ask for none
    assert ss.subspec_qlinear_plan(37, 37888, 3584, 4, 128)["workspace_bytes"] == 0
    assert ss.subspec_qlinear_plan(128, 7168, 5120, 3, 128)["workspace_bytes"] == 0
    assert ss.subspec_qlinear_plan(128, 37888, 3584, 4, 128)["workspace_bytes"] == 65536 + 128 * 28 * 4
    assert ss.subspec_qlinear_plan(8, 512, 256, 4, 64, ss.SUBSPEC_PATH_GEMV)["path"] == ss.SUBSPEC_PATH_GEMV
    assert ss.subspec_qlinear_plan(8, 512, 256, 4, 64, ss.SUBSPEC_PATH_MFMA)["path"] == ss.SUBSPEC_PATH_MFMA


def test_mfma_tile_shape_choice():
    """The automatic plan runs 32x32x16 tiles from M = 33 where 256-column groups of
    eight wavefronts (a four-chunk ring) cover at least half the 256 CUs and K is not
    split: 64 rows up to M = 64, 128 above (there, under three quarters of the CUs, groups
    of 64 take four wavefronts and two chunks and groups of 128 96 rows up to M = 96); and on a K of at least 128 blocks, two
    teams of four wavefronts per workgroup (the last tuple entry is then minus the
    wavefronts of one team; four chunks on 64 rows, two on 128).  Narrower launches run
    32-row tiles in row blocks while those stay within a workgroup per CU; everything
    else stays on 16x16x32 tiles."""
    def shape(M, N, K, bits=3, group=128, path=ss.SUBSPEC_PATH_AUTO):
        p = ss.subspec_qlinear_plan(M, N, K, bits, group, path)
        return p["mfma_rows"], p["rows"], p["ring_chunks"], p["waves"] // p["teams"] * (1 if p["teams"] == 1 else -1)
    assert shape(128, 55296, 5120) == (32, 128, 4, 8)      # 32B gate|up
    assert shape(128, 55296, 5120, 2, 64) == (32, 128, 4, 8)
    assert shape(128, 55296, 5120, 4, 128) == (32, 128, 4, 8)
    assert shape(128, 55296, 5120, 3, 64) == (32, 128, 4, 8)
    assert shape(97, 37888, 3584, 4) == (32, 128, 4, 8)     # 7B gate|up: 148 groups of 256
    assert shape(96, 37888, 3584, 4) == (32, 96, 4, 8)      # 96 rows up to M = 96
    assert shape(96, 49152, 3584, 4) == (32, 128, 4, 8)     # three quarters of the CUs: 128
    assert shape(96, 37888, 3584, 4, 64) == (32, 128, 2, 4)  # groups of 64: four wavefronts
    assert shape(128, 5120, 27648) == (32, 128, 2, -4)     # 32B down: two teams of four
    assert shape(96, 3584, 18944, 4) == (32, 128, 2, -4)   # 7B down
    assert shape(128, 7168, 5120) == (32, 32, 4, -4)  # 32B q|k|v: 32-row tiles
    assert shape(128, 14336, 4096, 4)[0] == 16       # more than a workgroup per CU
    assert shape(64, 55296, 5120) == (32, 64, 4, 8)        # 32B gate|up, 64-row tiles
    assert shape(33, 55296, 5120, 2, 64) == (32, 64, 4, 8)
    assert shape(48, 55296, 5120, 4, 128) == (32, 64, 4, 8)
    assert shape(32, 55296, 5120)[0] == 16
    assert shape(64, 37888, 3584, 4) == (32, 64, 4, 8)     # 7B gate|up: half-wide
    assert shape(33, 37888, 3584, 4) == (32, 64, 4, 8)
    assert shape(32, 37888, 3584, 4)[0] == 16
    assert shape(47, 44032, 256)[0] == 16 and shape(48, 44032, 256) == (32, 64, 4, 8)  # short K
    for N, rows in ((32768, 16), (32784, 32), (40960, 32), (40976, 16)):  # a tail of up to 64 column groups
        assert shape(47, N, 256)[0] == rows and shape(33, N, 128)[0] == 16, N
    assert shape(128, 55296, 512, 4, 64) == (32, 128, 2, 4)   # short K, no split tail: four wavefronts
    assert shape(128, 49152, 512, 4, 64) == (32, 128, 4, 8)
    assert shape(128, 49152, 128, 4, 64) == (32, 128, 2, 4)
    assert shape(128, 55296, 640, 4, 64) == (32, 128, 4, 8)
    assert shape(64, 5120, 27648) == (32, 64, 4, -4)       # long K: 64-row tiles on two teams
    assert shape(33, 3584, 18944, 4) == (32, 64, 4, -4)
    assert shape(32, 5120, 27648)[0] == 16
    assert shape(64, 7168, 5120) == (32, 32, 4, -4)        # q|k|v
    assert shape(64, 4608, 3584, 4)[0] == 16               # K under 36 blocks
    assert shape(17, 512, 256, path=ss.SUBSPEC_PATH_MFMA32) == (32, 128, 4, 4)
    # launches whose column groups number fewer than the CUs, with K under 128 blocks, run
    # their rows in blocks from M = 33 (q|k|v, o); long-K, wide and M <= 32 launches, keep one
    def blocks(M, N, K, bits=3, group=128):
        p = ss.subspec_qlinear_plan(M, N, K, bits, group)
        return p["row_blocks"], p["rows"]
    assert blocks(64, 7168, 5120) == (2, 32)              # 32B q|k|v
    assert blocks(128, 5120, 5120) == (4, 32)             # 32B o
    assert blocks(33, 4608, 3584, 4) == (2, 32)           # 7B q|k|v
    assert blocks(100, 3584, 3584, 4) == (4, 32)          # 7B o
    def blocks16(M, N, K, bits=3, group=128):
        p = ss.subspec_qlinear_plan(M, N, K, bits, group, ss.SUBSPEC_PATH_MFMA16)
        return p["mfma_rows"], p["row_blocks"], p["rows"]
    assert blocks16(64, 7168, 5120) == (16, 2, 32)
    assert blocks16(128, 5120, 5120) == (16, 2, 64)
    assert blocks16(100, 3584, 3584, 4) == (16, 2, 64)
    # a single k-block, and a K long enough to show the CUs left without work, keep two
    # 16x16x32 blocks
    assert blocks(128, 4608, 128, 4) == (2, 64) and blocks(128, 4608, 256, 4) == (4, 32)
    assert blocks(128, 5120, 9216) == (2, 64) and blocks(128, 5120, 9088) == (4, 32)
    assert blocks(97, 5376, 5248) == (2, 64) and blocks(97, 5376, 5120) == (4, 32)
    assert blocks(128, 5120, 16256, 2, 64) == (4, 32)
    assert blocks(97, 5376, 8320, 2, 64) == (2, 64) and blocks(97, 5376, 8192, 2, 64) == (4, 32)
    # the tail of 256-column groups is split where K is long for the rows
    for M, K, full in [(128, 2048, 0), (128, 2176, 256), (66, 1280, 0), (66, 1408, 256)]:
        assert ss.subspec_qlinear_plan(M, 69792, K, 4, 128)["full_groups"] == full, (M, K)
    assert blocks(96, 5120, 6144) == (3, 32) and blocks(128, 6144, 6144) == (4, 32)
    assert blocks(32, 7168, 5120) == (1, 32)
    assert blocks(64, 5120, 27648) == (1, 64)             # long K
    assert blocks(64, 3584, 18944, 4) == (1, 64)
    assert blocks(40, 37888, 3584, 4) == (1, 64)          # 592 column groups
    assert shape(128, 55296, 5120, path=ss.SUBSPEC_PATH_MFMA16)[0] == 16
    for path in (ss.SUBSPEC_PATH_MFMA16, ss.SUBSPEC_PATH_MFMA32):
        assert ss.subspec_qlinear_plan(40, 512, 256, 4, 64, path)["path"] == ss.SUBSPEC_PATH_MFMA


@pytest.mark.parametrize("tune,shape,expect", [
    ("mma_shape=16", (128, 7168, 5120, 3, 128), dict(mfma_rows=16, row_blocks=2)),
    ("mma_shape=16", (40, 37888, 3584, 4, 128), dict(mfma_rows=16)),
    ("row_split=2", (128, 7168, 5120, 3, 128), dict(mfma_rows=16, row_blocks=1)),
    ("rb_splits=-1", (128, 7168, 5120, 3, 128), dict(mfma_rows=16, row_blocks=2)),
    ("splits=3", (128, 7168, 5120, 3, 128), dict(mfma_rows=32, splits=3)),
    ("splits=2", (1, 4608, 3584, 4, 128), dict(splits=2)),  # not the small-batch launch
    ("mma8_half_min_m=48", (40, 37888, 3584, 4, 128), dict(mfma_rows=16)),
    # no such build (two-chunk rings of four wavefronts exist for groups of 64 only): the
    # four-chunk one, or the general choice
    ("mma_waves=4", (128, 55296, 5120, 3, 128), dict(mfma_rows=32, waves=4, ring_chunks=4)),
    ("mma_waves=4", (40, 3584, 18944, 4, 128), dict(mfma_rows=32, waves=8, teams=2, rows=64, ring_chunks=4)),
    ("mfma_pf=2", (40, 3584, 18944, 4, 64), dict(rows=128, waves=4, ring_chunks=2)),
    ("stream_nt=2,stream_ks=4", (6, 4608, 3584, 4, 128), dict(teams=1)),
])
def test_tuning_overrides_are_honoured(tune, shape, expect):
    """Measurement overrides reach the launch, and never one that was not built."""
    code = ("import paper_2509_18344_amd as ss, json; print(json.dumps(ss.subspec_qlinear_plan(*%r)))" % (shape,))
    out = subprocess.run([sys.executable, "-c", code], env=dict(os.environ, SUBSPEC_TUNE=tune), text=True,
                         capture_output=True, timeout=120, cwd=ROOT)
    assert out.returncode == 0, out.stderr
    plan = json.loads(out.stdout)
    assert {k: plan[k] for k in expect} == expect, plan


def test_gemv_plan_refuses_splits_longer_than_its_staging():
    # At 8 rows a GEMV split stages at most 2048 k of x.  With more than 16384 column
    # groups (N > 2^20) the plan cannot split K (one completion counter per group), so
    # K = 2560 would leave 512 k unstaged: refused, never silently wrong.
    N = (1 << 20) + 64
    with pytest.raises(ss.SubspecError, match="EUNSUPPORTED"):
        ss.subspec_qlinear_plan(8, N, 2560, 4, 128, ss.SUBSPEC_PATH_GEMV)
    assert "GEMV" in ss.subspec_last_error()
    # the same shape with K inside one staged span, and the MFMA path, still plan
    p = ss.subspec_qlinear_plan(8, N, 2048, 4, 128, ss.SUBSPEC_PATH_GEMV)
    assert p["splits"] == 1
    assert ss.subspec_qlinear_plan(8, N, 2560, 4, 128, ss.SUBSPEC_PATH_MFMA)["splits"] >= 1
    # below the counter limit the plan splits K instead
    p = ss.subspec_qlinear_plan(8, 65536, 8192, 4, 128, ss.SUBSPEC_PATH_GEMV)
    assert p["splits"] * p["blocks_per_split"] * 128 >= 8192 and p["blocks_per_split"] * 128 <= 2048


def test_noalloc_refuses_shapes_beyond_its_fixed_scratch():
    # 32x32 kernel at M = 128 over K = 4325376 with groups of 64: the sums of x alone
    # (128 x 67584 fp32) exceed the 32 MiB array, so even an unsplit plan cannot fit;
    # the call is refused while planning, before any GPU work
    assert ss.SUBSPEC_NOALLOC_SCRATCH_BYTES == 32 << 20
    with pytest.raises(ss.SubspecError, match="EUNSUPPORTED"):
        ss.subspec_qlinear_noalloc(16, 16, 16, 16, 4, 64, 128, 256, 4325376, 16, stream=0)
    assert "scratch" in ss.subspec_last_error()


def test_qlinear_argument_errors_need_no_gpu():
    with pytest.raises(ss.SubspecError) as ei:
        ss.subspec_qlinear(None, 16, 16, 16, 4, 64, 1, 512, 256, 16, stream=0)
    assert "EINVAL" in str(ei.value) and "null" in ss.subspec_last_error()
    with pytest.raises(ss.SubspecError) as ei:
        ss.subspec_qlinear(16, 16, 16, 24, 4, 64, 1, 512, 256, 16, stream=0)
    assert "aligned" in ss.subspec_last_error()
    with pytest.raises(ss.SubspecError):
        ss.subspec_qlinear_path(16, 16, 16, 16, 4, 64, 9, 512, 256, 16, ss.SUBSPEC_PATH_GEMV, stream=0)
    with pytest.raises(ss.SubspecError):
        ss.subspec_quantize(16, 4, 64, 16, 100, 16, 16, 16, stream=0)


def test_current_stream_without_torchs_private_names(monkeypatch):
    """The current stream comes from torch's public Stream object where the private names
    that give its handle directly are missing."""
    import types
    fake = types.SimpleNamespace(
        _C=types.SimpleNamespace(),
        cuda=types.SimpleNamespace(is_initialized=lambda: True,
                                   current_stream=lambda: types.SimpleNamespace(cuda_stream=0x5150)))
    monkeypatch.setitem(sys.modules, "torch", fake)
    monkeypatch.setattr(_binding, "_torch", None)
    for n in ("_raw_stream", "_device"):
        monkeypatch.setattr(_binding, n, None, raising=False)
    assert _binding._stream(None) == 0x5150
    # and through them where they are there
    fake._C._cuda_getCurrentRawStream, fake._C._cuda_getDevice = lambda d: 0x1000 + d, lambda: 3
    monkeypatch.setattr(_binding, "_torch", None)
    assert _binding._stream(None) == 0x1003


def test_binding_fails_loudly_without_library(monkeypatch, tmp_path):
    monkeypatch.setattr(_binding, "_lib", None)
    monkeypatch.setattr(_binding, "_HERE", str(tmp_path))
    with pytest.raises(RuntimeError, match="missing"):
        _binding.load_library()


def test_tree_expand_argument_errors_need_no_gpu():
    # (R, V, k, T): rejected before any GPU work
    for R, V, k, T, err in [(0, 64, 1, 0.2, "EUNSUPPORTED"), (1025, 64, 1, 0.2, "EUNSUPPORTED"),
                            (2, 100, 1, 0.2, "EUNSUPPORTED"), (2, 64, 0, 0.2, "EUNSUPPORTED"),
                            (2, 64, 33, 0.2, "EUNSUPPORTED"), (1, 8, 9, 0.2, "EUNSUPPORTED"),
                            (2, 64, 4, 0.0, "EINVAL"), (2, 64, 4, -1.0, "EINVAL"),
                            (1000, 1 << 22, 4, 0.2, "EUNSUPPORTED")]:
        with pytest.raises(ss.SubspecError) as ei:
            ss.subspec_tree_expand(16, 16, R, V, T, k, 16, 16, 16, stream=0)
        assert err in str(ei.value), (R, V, k, T)
    with pytest.raises(ss.SubspecError):
        ss.subspec_tree_expand(None, 16, 2, 64, 0.2, 4, 16, 16, 16, stream=0)
    with pytest.raises(ss.SubspecError):
        ss.subspec_tree_expand(24, 16, 2, 64, 0.2, 4, 16, 16, 16, stream=0)
    assert ss.subspec_tree_workspace_bytes(6, 152064, 6) > 65536
    assert ss.subspec_tree_workspace_bytes(6, 100, 6) == 0


def test_tree_plan_shapes():
    # the launch's own slices: at most 256 workgroups up to 32 rows (16 with lists of 32),
    # at most 512 up to 128 and about as many beyond, each at least 2048 logits (one 16-byte load per thread) unless the row is shorter;
    # slices are multiples of 8 and cover the row
    assert ss.subspec_tree_plan(6, 152064, 6) == (42, 3624, 8)
    assert ss.subspec_tree_plan(64, 152064, 6) == (8, 19008, 8)
    assert ss.subspec_tree_plan(1, 152064, 6) == (75, 2032, 8)
    assert ss.subspec_tree_plan(1024, 64, 32) == (1, 64, 32)
    assert ss.subspec_tree_plan(37, 4096, 17) == (2, 2048, 32)
    assert ss.subspec_tree_plan(3, 2048, 9)[2] == 16
    for R in range(1, 129):
        for k in (1, 6, 8, 16, 17, 32):
            c, n, _ = ss.subspec_tree_plan(R, 152064, k)
            # what the threads of the second phase hold in registers at k <= 8: two lists each
            assert R * c <= (256 if R <= 16 or (R <= 32 and k <= 16) else 512), (R, k, c)
    assert ss.subspec_tree_plan(33, 152064, 6) == (15, 10144, 8)
    assert ss.subspec_tree_plan(32, 152064, 32) == (16, 9504, 32)
    assert ss.subspec_tree_plan(171, 152064, 6)[0] == 3 and ss.subspec_tree_plan(171, 152064, 32)[0] == 2
    for R, V, k in [(1, 8, 1), (6, 1000, 6), (128, 152064, 6), (1000, 2048, 32), (7, 152064, 16)]:
        c, n, _ = ss.subspec_tree_plan(R, V, k)
        assert n % 8 == 0 and (c - 1) * n < V <= c * n and R * c <= 1024, (R, V, k)
        # the workspace holds the launch's lists: completion counters, then per workgroup
        # a (max, sum) pair and k (score, token) pairs
        assert ss.subspec_tree_workspace_bytes(R, V, k) == 65536 + R * c * 8 * (1 + k)
    for R, V, k in [(0, 64, 1), (2, 100, 1), (2, 64, 33), (1, 8, 9)]:
        with pytest.raises(ss.SubspecError, match="EUNSUPPORTED"):
            ss.subspec_tree_plan(R, V, k)


def test_tree_attention_plan_and_errors_need_no_gpu():
    # Qwen2.5-7B at the last pass of a depth-48 tree: 2336 keys = 73 tiles of 32,
    # three tiles per range
    assert ss.subspec_tree_attention_plan(6, 28, 4, 2048, 282) == (25, 3)
    for M, Hq, Hkv, P, T in [(6, 28, 4, 0, 0), (1, 1, 1, 0, 0), (6, 40, 8, 30000, 282), (8, 16, 2, 33, 7)]:
        s, t = ss.subspec_tree_attention_plan(M, Hq, Hkv, P, T)
        tiles = -(-(P + T + M) // 32)
        assert t >= 1 and (s - 1) * t < tiles <= s * t, (M, Hq, Hkv, P, T)
        rows_pad = 16 * -(-(Hq // Hkv * M) // 16)
        # the split-K completion counters (64 KiB) stay in front of the partials
        assert ss.subspec_tree_attention_workspace_bytes(M, Hq, Hkv, P, T) == \
            65536 + Hkv * s * rows_pad * (128 + 2) * 4
    for M, Hq, Hkv, P, T in [(6, 30, 4, 10, 0), (0, 28, 4, 10, 0), (10, 28, 4, 10, 0), (6, 28, 4, -1, 0),
                             (64, 1, 1, 0, 1100), (6, 4, 0, 10, 0)]:
        with pytest.raises(ss.SubspecError, match="EUNSUPPORTED"):
            ss.subspec_tree_attention_plan(M, Hq, Hkv, P, T)
        assert ss.subspec_tree_attention_workspace_bytes(M, Hq, Hkv, P, T) == 0
    args = dict(M=6, Hq=28, Hkv=4, S=2400, P=2048, T=282, scale=0.088)

    def call(q=16, kc=16, vc=16, kn=16, vn=16, mask=16, out=16, **kw):
        a = dict(args, **kw)
        return ss.subspec_tree_attention(q, kc, vc, kn, vn, mask, a["M"], a["Hq"], a["Hkv"], a["S"], a["P"],
                                         a["T"], a["scale"], out, stream=0)
    with pytest.raises(ss.SubspecError, match="EINVAL"):
        call(q=None)
    with pytest.raises(ss.SubspecError, match="EINVAL"):
        call(kc=24)
    with pytest.raises(ss.SubspecError, match="EINVAL"):
        call(mask=18)
    with pytest.raises(ss.SubspecError, match="EUNSUPPORTED"):
        call(S=2335)
    with pytest.raises(ss.SubspecError, match="EINVAL"):
        call(scale=float("inf"))


def test_prefetch_argument_errors_need_no_gpu():
    for slot_bytes, slots in [(0, 2), (1024, 1), (1024, 65)]:
        with pytest.raises(ss.SubspecError, match="EINVAL"):
            ss.Prefetcher(slot_bytes, slots)
    lib = ss.load_library()
    import ctypes
    t = ctypes.c_longlong()
    p = ctypes.c_void_p()
    assert lib.subspec_prefetch_begin(None, None, 16, ctypes.byref(t)) == -1  # SUBSPEC_EINVAL
    assert lib.subspec_prefetch_acquire(None, 0, None, ctypes.byref(p)) == -1  # SUBSPEC_EINVAL
    assert lib.subspec_prefetch_release(None, 0, None) == -1  # SUBSPEC_EINVAL
    assert lib.subspec_prefetch_destroy(None) == -1  # SUBSPEC_EINVAL
    assert lib.subspec_prefetch_create(16, 2, None) == -1  # SUBSPEC_EINVAL


def test_quantize_hqq_argument_errors_need_no_gpu():
    with pytest.raises(ss.SubspecError, match="EUNSUPPORTED"):
        ss.subspec_quantize_hqq(16, 5, 64, 16, 128, 16, 16, 16, stream=0)
    with pytest.raises(ss.SubspecError, match="EINVAL"):
        ss.subspec_quantize_hqq(16, 4, 64, 16, 100, 16, 16, 16, stream=0)
    with pytest.raises(ss.SubspecError, match="EINVAL"):
        ss.subspec_quantize_hqq(None, 4, 64, 16, 128, 16, 16, 16, stream=0)
    with pytest.raises(ss.SubspecError, match="EINVAL"):
        ss.subspec_quantize_hqq(16, 4, 64, 16, 128, 24, 16, 16, stream=0)
