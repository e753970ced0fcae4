"""Host-side checks that need no GPU: the shared library loads, exports every
symbol the public header declares, and rejects bad arguments before launching
anything."""
import ctypes
import os
import random
import re

import numpy as np
import pytest
import torch

from paper_2504_14152_amd import build, fgmp

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _declared_symbols():
    text = open(os.path.join(ROOT, "include", "fgmp.h")).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    return sorted(set(re.findall(r"\b(fgmp_[a-z_0-9]+)\s*\(", text)))


def test_library_exports_every_declared_symbol():
    if not os.path.exists(build.lib_path()):
        build.build()
    lib = ctypes.CDLL(build.lib_path())
    names = _declared_symbols()
    assert {"fgmp_quantize_weights", "fgmp_quantize_activations", "fgmp_gemm", "fgmp_quant_gemm_fused",
            "fgmp_unpack_canonical"} <= set(names)
    for name in names:
        assert hasattr(lib, name), f"{name} declared in fgmp.h but not exported"


def test_sizes_and_host_side_argument_checks():
    assert fgmp.version().endswith("(gfx950)")
    # 8 x 128 tiles: header + 512 B + 64 B + 8 B + 4 B + 512 B per tile, planes 256-byte aligned
    assert fgmp.packed_bytes(8, 128) == 256 + 512 + 256 + 256 + 256 + 512
    assert fgmp.packed_bytes(8, 24) == 0 and fgmp.packed_bytes(0, 16) == 0
    n_blocks = 4096 * 4096 // 16
    # worst case: 8 + 8 B values, the scale-or-index byte, 1 mask bit, 4 B of tile table per 64 blocks
    assert 16.125 * n_blocks <= fgmp.packed_bytes(4096, 4096) <= (17 + 0.125 + 0.0625) * n_blocks + 2048
    assert fgmp.workspace_bytes(4096, 12288, 4096) >= fgmp.packed_bytes(4096, 4096)
    L = fgmp.lib()
    assert L.fgmp_quantize_activations(None, 0, 8, 128, 128, None, 0.0, 1.0, None, 0, None, None) == -1
    # measurement helper: no sink, no work
    assert L.fgmp_selftest_mfma_rate(256, 10, None, None) == -1
    # measurement hook: a lone event is refused, clearing always works
    assert L.fgmp_selftest_time_gemm_kernel(256, None) == -1
    assert L.fgmp_selftest_time_gemm_kernel(None, None) == 0
    assert L.fgmp_gemm(None, 1, None, 1, 16, None, 1, None, 0, None) == -1
    assert L.fgmp_gemm(256, 1, 256, 1, 24, 256, 1, 256, 0, None) == -2
    assert L.fgmp_unpack_canonical(None, 1, 16, None, None, None, None) == -1
    # the entry points added for the score of Eq. 8, clipping, packed output and the global threshold
    assert L.fgmp_quantize_activations_ex(256, 0, 8, 128, 128, 256, 0.0, 1.0, 5, 256, 1 << 20, None, None) == -1
    assert L.fgmp_quantize_weights_ex(None, 0, 8, 128, 128, None, 0, 0.0, 1.0, 1, None, 0, None, None) == -1
    assert L.fgmp_quantize_weights_clip(256, 0, 8, 128, 128, 256, 0, 0.0, 1.0, 256, 1 << 20, None, None, 0, None) == -1
    assert L.fgmp_quantize_weights_clip(256, 0, 8, 24, 24, 256, 0, 0.0, 1.0, 256, 1 << 20, None, 256, 64, None) == -2
    assert L.fgmp_quantize_weights_clip(256, 0, 8, 128, 128, 256, 0, 0.0, 1.0, 256, 1 << 20, None, 256, 63, None) == -4
    assert fgmp.lib().fgmp_workspace_bytes_packed_out(4096, 12288, 4096) >= fgmp.workspace_bytes(4096, 12288, 4096) + 4096 * 12288 * 4
    assert fgmp.lib().fgmp_workspace_bytes_packed_out(64, 24, 128) == 0          # N must be a multiple of 16
    # gated epilogue: groups of 64 weight rows, no room beyond the plain one's (the gate is applied as the product is read), known operators only
    wb = fgmp.lib().fgmp_workspace_bytes_packed_out_ex
    assert wb(64, 96, 128, 1) == 0 and wb(64, 128, 128, 7) == 0
    assert wb(64, 128, 128, 0) == fgmp.lib().fgmp_workspace_bytes_packed_out(64, 128, 128)
    assert wb(64, 128, 128, 1) == wb(64, 128, 128, 0) and wb(2048, 22016, 4096, 1) == wb(2048, 22016, 4096, 0)
    # the one-launch flag changes no size and is no operator of its own
    assert wb(8, 12288, 4096, 0x100) == wb(8, 12288, 4096, 0) and wb(64, 128, 128, 0x101) == wb(64, 128, 128, 1)
    assert wb(64, 128, 128, 0x102) == 0 and wb(64, 128, 128, 0x200) == 0
    # ... and a decode step's workspace has room for its row groups' decision words behind its own scratch
    assert wb(8, 12288, 4096, 0x100) >= fgmp.workspace_bytes(8, 12288, 4096) + 12288 // 16 * 4
    assert L.fgmp_quant_gemm_fused_packed_out_ex(256, 0, 64, 128, 128, 256, 0.0, 1.0, 256, 96, 1, 256, 0.0, 1.0, 256, 1 << 20,
                                                 None, 256, 1 << 30, None) == -2
    assert L.fgmp_quant_gemm_fused_packed_out_ex(256, 0, 64, 128, 128, 256, 0.0, 1.0, 256, 128, 5, 256, 0.0, 1.0, 256, 1 << 20,
                                                 None, 256, 1 << 30, None) == -1
    assert L.fgmp_quant_gemm_fused_packed_out(256, 0, 64, 128, 128, 256, 0.0, 1.0, 256, 24, 256, 0.0, 1.0, 256, 1 << 20,
                                              None, 256, 1 << 20, None) == -2
    assert L.fgmp_quant_gemm_fused_packed_out(256, 0, 64, 128, 128, 256, 0.0, 1.0, 256, 32, 256, 0.0, 0.0, 256, 1 << 20,
                                              None, 256, 1 << 20, None) == -1   # output scale must be positive
    assert L.fgmp_quant_gemm_fused_packed_out(256, 0, 64, 128, 128, 256, 0.0, 1.0, 256, 32, 256, 0.0, 1.0, 256, 16,
                                              None, 256, 1 << 20, None) == -4   # packed output buffer too small
    assert L.fgmp_threshold_for_fraction_multi(None, None, 1, ctypes.c_double(0.1), None, None) == -1
    # the quantizer's traffic model exists in measurement builds only
    assert L.fgmp_selftest_quantizer_traffic(256, 0, 16384, 8192, 8192, 256, 256, 1 << 30, None) == -5


def test_bench_refuses_more_than_one_gpu():
    import subprocess
    import sys
    res = subprocess.run([sys.executable, os.path.join(ROOT, "bench.py"), "--gpus", "2"], capture_output=True, text=True)
    assert res.returncode != 0 and "one GPU" in res.stderr


def test_workspace_sizes_over_the_row_counts_where_the_paths_change():
    """Host-side planning only: every M from decode sizes through the first prefill tiles gets a workspace,
    whichever kernel the planner picks (decode steps, mid-size products, tiles split along K, whole tiles), and it never
    shrinks below what the FP16 copy of X alone needs."""
    L = fgmp.lib()
    for (N, K) in [(12288, 4096), (4096, 4096), (22016, 4096), (4096, 11008), (264, 2048), (57344, 8192)]:
        for M in list(range(1, 300)) + [511, 512, 513, 1024, 4096]:
            ws = int(L.fgmp_workspace_bytes(M, N, K))
            assert ws >= M * K * 2, (M, N, K, ws)
            assert ws < (1 << 34), (M, N, K, ws)
        assert L.fgmp_workspace_bytes(0, N, K) == 0 and L.fgmp_workspace_bytes(8, N, K + 8) == 0


def test_a_workspace_for_a_large_batch_serves_the_smaller_ones():
    """A server allocates once, for its largest batch: above 32 rows a size is never below that of 32 or fewer rows, nor --
    within one row of 256 x 256 tiles -- below that of fewer rows, plain and with packed results, whichever kernel each takes."""
    L = fgmp.lib()
    for (N, K) in [(12288, 4096), (4096, 4096), (22016, 4096), (4096, 11008), (264, 2048), (57344, 8192), (16384, 512), (64, 65536)]:
        rows = list(range(1, 33)) + [33, 48, 64, 100, 128, 192, 200, 224, 256, 257, 300, 384, 448, 512, 513, 768, 1024, 1025, 2048, 4096]
        plain = [int(L.fgmp_workspace_bytes(M, N, K)) for M in rows]
        for sizes in (plain, [int(L.fgmp_workspace_bytes_packed_out_ex(M, N, K, 0)) for M in rows] if N % 16 == 0 else plain,
                      [int(L.fgmp_workspace_bytes_packed_out_ex(M, N, K, 1)) for M in rows] if N % 64 == 0 else plain):
            for i, M in enumerate(rows):
                for j in range(i):
                    if M > 32 and (rows[j] <= 32 or (rows[j] - 1) // 256 == (M - 1) // 256):
                        assert sizes[i] >= sizes[j], (M, rows[j], N, K)


def test_the_mid_size_shapes_cover_every_arrangement_the_planner_uses():
    """The GPU tests name the arrangement each shape is meant for; over the kernel's whole range the planner uses no other
    (16-row groups 2 to 8, column groups 2 to 4 up to 4 of them and 2 to 3 above)."""
    import random
    from tests.test_gpu_size_edges import MID_PLANS
    named = set()
    for (M, K, N), groups, shared in MID_PLANS:
        route = fgmp.selftest_gemm_route(M, N, K)
        assert route[0] == 2 and route[1:3] == groups and (route[5] > 1) == shared, ((M, K, N), route)
        named.add((groups, shared))
    rng = random.Random(7)
    seen = set()
    for _ in range(60000):
        r = fgmp.selftest_gemm_route(rng.choice((rng.randint(20, 1024), rng.randint(1025, 4096))), int(2 ** rng.uniform(3, 16)), 16 * int(2 ** rng.uniform(0, 11)))
        if r[0] == 2:
            seen.add((r[1:3], r[5] > 1))
    assert len(seen) > 20 and seen <= named, seen - named
    # 33 to 1024 rows of the Llama-2-7B linears, and what the neighbours of the range take
    assert [fgmp.selftest_gemm_route(M, 12288, 4096)[0] for M in (1, 32, 33, 64, 4096)] == [0, 0, 2, 2, 3]
    # up to 32 rows: one launch where a workgroup has one round of row groups, whatever the length
    assert [fgmp.selftest_gemm_route(M, 4096, 11008)[0] for M in (20, 24, 28, 32)] == [2, 2, 0, 0]
    assert [fgmp.selftest_gemm_route(M, 11008, 5120)[0] for M in (20, 26, 28, 32)] == [0, 0, 2, 2]
    assert fgmp.selftest_gemm_route(19, 24, 32768)[0] == 1 and fgmp.selftest_gemm_route(32, 264, 32768)[0] == 2
    assert fgmp.lib().fgmp_selftest_gemm_route(8, 24, 24, (ctypes.c_int64 * 6)()) == -2
    assert fgmp.lib().fgmp_selftest_gemm_route(8, 24, 16, None) == -1


def test_long_products_of_few_columns_keep_the_mid_size_kernel_within_their_workspace():
    """Sums of K in many parts can need more than the prefill kernel does: fewer parts then, not another kernel; and what the static
    scratch array serves on the prefill kernel it serves with them."""
    L = fgmp.lib()
    for (M, K, N) in [(695, 7808, 394), (260, 10224, 16566), (497, 9744, 385), (744, 6960, 491), (609, 10160, 12095), (449, 8816, 486)]:
        route = fgmp.selftest_gemm_route(M, N, K)
        assert route[0] == 2, ((M, K, N), route)
        mp = -(-M // 256) * 256
        assert L.fgmp_workspace_bytes(M, N, K) <= L.fgmp_workspace_bytes(mp, N, K)
        tiles = mp // 256 * -(-N // 256) % 256           # of a last round: FP32 sums of four parts, or two
        fused = mp * (-(-K // 128) * 128) * 2 + (0 if tiles > 128 else tiles * (2 if tiles > 64 else 6) << 18)
        if fused + 65536 + 4096 <= fgmp.STATIC_SCRATCH_BYTES:
            too_small = -4                                # FGMP_ERR_BUFFER_TOO_SMALL, decided before the arguments are looked at
            assert L.fgmp_quant_gemm_fused_static_scratch(None, 0, M, K, K, None, 0.0, 1.0, None, N, None, N, None) != too_small


def test_estimates_decide_above_1024_rows_as_below():
    for (M, K, N) in [(1100, 512, 264), (1300, 1040, 512), (1300, 768, 2048), (1100, 1040, 3400), (1025, 512, 4096)]:
        assert [fgmp.selftest_gemm_route(m, N, K)[0] for m in (1024, M, 1301)] == [2, 2, 2], (M, K, N)


def test_an_odd_number_of_row_tiles_takes_the_kernel_of_its_even_neighbours():
    """20 to 32 rows, long products; where the neighbours differ, the estimates are next to each other."""
    for (M, K, N) in [(20, 5120, 11000), (20, 8192, 8184), (32, 11008, 4088), (24, 11008, 4088), (28, 5120, 11000), (20, 4096, 22008)]:
        near = {fgmp.selftest_gemm_route(M, n, K)[0] for n in (N - 8, N + 8)}
        assert -(-N // 8) % 2 == 1 and near == {fgmp.selftest_gemm_route(M, N, K)[0]}, (M, K, N)
    assert fgmp.selftest_gemm_route(20, 8184, 8192)[0] == 0 and fgmp.selftest_gemm_route(24, 4088, 11008)[0] == 2


def test_the_first_workgroups_quantize_for_all():
    """Products of 33 rows on that quantize in their launch: where the chip does not hold two such launches, no more workgroups hold a
    share than it takes at four pieces of 64 blocks each (dealt out over all of them, overlapping launches wait for workgroups that
    have not started), and never more than eight pieces, one per wave, fall to one."""
    rng = random.Random(5)
    seen = 0
    for M, K, N in [(64, 4096, 12288), (77, 2064, 5003), (200, 4096, 22016), (512, 4096, 4096), (33, 160, 16503)] + [
            (int(2 ** rng.uniform(5.1, 10)), 16 * int(2 ** rng.uniform(0, 9.5)), int(2 ** rng.uniform(3, 14.5))) for _ in range(400)]:
        route = fgmp.selftest_gemm_route(M, N, K)
        holders = fgmp.selftest_quantizing_workgroups(M, N, K)
        workgroups, pieces = route[3] * route[4] * route[5], -(-M * 8 * -(-K // 128) // 64)
        in_launch = route[0] == 2 and workgroups <= 256 and M * 8 * -(-K // 128) <= 512 * workgroups
        assert holders == (min(workgroups, pieces if workgroups <= 128 else -(-pieces // 4)) if in_launch else 0), (M, K, N)
        if in_launch:
            seen += 1
            assert pieces <= 8 * holders
    assert seen >= 100
    assert fgmp.lib().fgmp_selftest_quantizing_workgroups(8, 24, 24) == -2 and fgmp.lib().fgmp_selftest_quantizing_workgroups(0, 24, 16) == -1


class _Pretend:
    """What the binding asks of a GPU tensor, without one."""
    is_cuda = True

    def __init__(self, at, shape, dtype=torch.float32, cuda=True):
        self.at, self.shape, self.dtype, self.is_cuda = at, torch.Size(shape), dtype, cuda

    def data_ptr(self):
        return self.at

    def stride(self, dim):
        return (self.shape[1] + 8, 1)[dim]

    def numel(self):
        return self.shape.numel()


@pytest.mark.parametrize("dtype,code", [(torch.float32, 0), (torch.bfloat16, 1)])
def test_the_extension_hands_on_what_it_is_given(dtype, code):
    got = []
    i64, f32, vp = ctypes.c_int64, ctypes.c_float, ctypes.c_void_p
    proto = ctypes.CFUNCTYPE(ctypes.c_int, vp, ctypes.c_int, i64, i64, i64, vp, f32, f32, vp, i64, vp, i64, vp, ctypes.c_size_t, vp)
    entry = proto(lambda *a: got.append(a) or -4)
    fgmp.lib()
    top = 1 << 47

    def call(X, f, T, S, w, Y, ws):
        return fgmp._call.quant_gemm_fused(ctypes.cast(entry, vp).value, torch.float32, torch.bfloat16, X, f, T, S, w, Y, ws, 0x77)

    X, f, Y = _Pretend(top + 16, (3, 32), dtype), _Pretend(top + 32, (32,)), _Pretend(top + 48, (3, 40))
    w, ws = fgmp.Packed(_Pretend(top + 64, (999,)), 40, 32), _Pretend(top + 80, (12345,))
    assert call(X, f, 0.25, np.float32(1.5), w, Y, ws) == -4
    assert got == [(top + 16, code, 3, 32, 40, top + 32, 0.25, 1.5, top + 64, 40, top + 48, 48, top + 80, 12345, 0x77)]
    # whatever the general path refuses, or takes in a way of its own, is left to it, and nothing is called
    bad = [(_Pretend(16, (3, 32), dtype, cuda=False), f, 0.25, 1.5, w, Y, ws), (X, _Pretend(32, (32,), cuda=False), 0.25, 1.5, w, Y, ws),
           (_Pretend(16, (3, 48), dtype), f, 0.25, 1.5, w, Y, ws), (_Pretend(16, (3, 32), torch.float16), f, 0.25, 1.5, w, Y, ws),
           (_Pretend(16, (32,), dtype), f, 0.25, 1.5, w, Y, ws), (X, f, None, 1.5, w, Y, ws), (X, f, 0.25, 1.5, w, "out", ws),
           (X, f, 0.25, 1.5, w, Y, None), (X, f, 0.25, 1.5, None, Y, ws)]
    assert [call(*b) for b in bad] == [None] * len(bad) and len(got) == 1


def test_without_a_c_compiler_the_binding_takes_ctypes(tmp_path, monkeypatch):
    """The extension module saves host time and nothing else: where it is not there and cannot be built, libraries load and every
    entry point works through ctypes."""
    monkeypatch.setattr(build, "CALL", str(tmp_path / "module.so"))
    monkeypatch.setenv("CC", str(tmp_path / "no-compiler"))
    monkeypatch.setattr(fgmp, "_call", None)
    fgmp._load_call.cache_clear()
    try:
        assert fgmp._load(build.lib_path()).fgmp_version() == fgmp.lib().fgmp_version() and fgmp._call is None
        monkeypatch.setattr(fgmp, "_stream", lambda: 0)
        X, f, w = _Pretend(16, (3, 48)), _Pretend(32, (48,)), fgmp.Packed(_Pretend(64, (999,)), 40, 32)
        with pytest.raises(fgmp.FgmpError, match="K mismatch"):   # (what the general path says)
            fgmp.quant_gemm_fused(X, f, 0.5, 1.0, w, out=_Pretend(48, (3, 40)), workspace=_Pretend(80, (12345,)))
    finally:
        fgmp._load_call.cache_clear()


def test_the_extension_is_this_interpreters_and_appears_whole(tmp_path, monkeypatch):
    """Named with the interpreter's tag, so that no other one loads it; compiled beside its place and moved there: who finds the file
    finds all of it, and a build that fails leaves what was there."""
    import sysconfig
    assert build.CALL.endswith(sysconfig.get_config_var("EXT_SUFFIX")) and "cpython" in os.path.basename(build.CALL)
    place = tmp_path / "module.so"
    place.write_text("before")
    compiler = tmp_path / "cc"
    compiler.write_text("#!/bin/sh\nwhile [ $# -gt 1 ]; do if [ $1 = -o ]; then out=$2; fi; shift; done\necho half > $out\ncp %s %s.seen\nexit $STATUS\n" % (place, place))
    compiler.chmod(0o755)
    monkeypatch.setattr(build, "CALL", str(place))
    monkeypatch.setenv("CC", str(compiler))
    monkeypatch.setenv("STATUS", "1")
    with pytest.raises(RuntimeError):
        build.build_call()
    assert place.read_text() == "before"
    monkeypatch.setenv("STATUS", "0")
    assert build.build_call() == str(place) and place.read_text() == "half\n"
    assert (tmp_path / "module.so.seen").read_text() == "before" and sorted(os.listdir(tmp_path)) == ["cc", "module.so", "module.so.seen"]


@pytest.mark.parametrize("what", ["X.is_cuda", "X.shape", "X.dtype", "X.data_ptr", "X.stride", "fisher.is_cuda", "fisher.data_ptr", "w.K", "w.rows",
                                  "w.buf.data_ptr", "out.data_ptr", "out.stride", "workspace.data_ptr", "workspace.numel"])
def test_the_extension_asks_nothing_more_once_something_failed(what):
    """An argument that raises ends it: no other object is asked with that exception pending, and the general path says what is wrong."""
    asked = []

    class Asked:
        def __init__(self, name, of):
            self._name, self._of = name, of

        def __getattr__(self, key):
            asked.append(f"{self._name}.{key}")
            if asked[-1] == what:
                raise ValueError(key)
            value = getattr(self._of, key)
            if key == "buf":
                return Asked(f"{self._name}.buf", value)
            return value

    fgmp.lib()
    proto = ctypes.CFUNCTYPE(ctypes.c_int)
    entry = proto(lambda: asked.append("called") or 0)
    X, f, Y, ws = (Asked(n, _Pretend(16, shape)) for n, shape in (("X", (3, 32)), ("fisher", (32,)), ("out", (3, 40)), ("workspace", (99,))))
    w = Asked("w", fgmp.Packed(_Pretend(64, (999,)), 40, 32))
    rc = fgmp._call.quant_gemm_fused(ctypes.cast(entry, ctypes.c_void_p).value, torch.float32, torch.bfloat16, X, f, 0.5, 1.0, w, Y, ws, 0)
    assert rc is None and asked[-1] == what and "called" not in asked
