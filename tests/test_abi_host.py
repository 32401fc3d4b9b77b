"""Host-side checks of the C ABI that need no GPU: the library loads, exports
every symbol the header declares, and rejects bad arguments before touching a
device."""
import ctypes
import os
import re
import subprocess
import sys

import pytest

from paper_2505_00232_amd import binding, build

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def L():
    if not os.path.exists(binding.LIB_PATH):
        build.build()
    return binding.lib()


def _declared(header_name):
    header = open(os.path.join(ROOT, "include", header_name)).read()
    return set(re.findall(r"\b(qfc_[a-z0-9_]+)\s*\(", header))


def test_header_symbols_are_exported(L):
    """qfc.h declares exactly the binding's entry points, and the library's dynamic symbol table
    holds no qfc_* function beyond what the two headers declare (qfc_experimental.h: the
    tunables of tests and sweeps, which are not part of the interface)."""
    declared = _declared("qfc.h")
    assert declared == set(binding.EXPORTS)
    for name in declared:
        assert hasattr(L, name), name
    experimental = _declared("qfc_experimental.h")
    assert experimental == {"qfc_tune", "qfc_probe_mfma"}
    nm = subprocess.run(["nm", "-D", "--defined-only", binding.LIB_PATH], capture_output=True, text=True, check=True)
    exported = {ln.split()[-1] for ln in nm.stdout.splitlines() if len(ln.split()) >= 3 and ln.split()[-2] in "TW"}
    assert {e for e in exported if e.startswith("qfc_")} == declared | experimental


def test_status_strings(L):
    seen = {binding.status_string(c) for c in range(7)}
    assert len(seen) == 7 and binding.status_string(0) == "ok"
    assert binding.status_string(99) == "unknown status"


def test_packed_size_and_descriptor_checks(L):
    d = binding.make_desc(1024, 512, "w8c")
    # 1024 x 512 codes + 1024 fp32 scales, no padding needed
    assert binding.qfc_packed_size(d) == 1024 * 512 + 4 * 1024
    d = binding.make_desc(4096, 2304, "w4g32")
    # per 16 rows: 18 KiB tiles of 128 k plus 3 scale tiles
    assert binding.qfc_packed_size(d) == (4096 // 16) * (18 + 3) * 1024
    d = binding.make_desc(1, 32, "w4g32")
    assert binding.qfc_packed_size(d) == 16 * 2 * 1024  # padded to 256 rows x 128 k, one scale tile each
    d = binding.make_desc(4096, 2304, "w4c")
    # per 16 rows: 18 KiB tiles of 128 k, no scale tiles; 4096 fp32 scales follow
    assert binding.qfc_packed_size(d) == (4096 // 16) * 18 * 1024 + 4 * 4096
    out = ctypes.c_size_t(0)
    bad = [binding.Desc(0, 512, 8, 0, 0, 1), binding.Desc(8, 48, 8, 0, 0, 1), binding.Desc(8, 64, 3, 0, 0, 1),
           binding.Desc(8, 64, 8, -1, 0, 1), binding.Desc(8, 64, 8, 0, 7, 1), binding.Desc(8, 64, 8, 0, 0, 5)]
    assert binding.qfc_packed_size(binding.Desc(8, 64, 4, 0, 0, 2)) > 0  # int8-activation decode, per-channel int4
    for d in bad:
        assert L.qfc_packed_size(ctypes.byref(d), ctypes.byref(out)) == 1
    assert binding.qfc_packed_size(binding.Desc(8, 64, 4, 0, 0, 1)) > 0  # int8-activation prefill, per-channel int4 ("8/4/4")
    unsupported = [binding.Desc(8, 64, 8, 32, 0, 1), binding.Desc(8, 64, 4, 32, 1, 1),
                   binding.Desc(8, 64, 4, 0, 1, 0), binding.Desc(8, 64, 8, 0, 1, 1),
                   binding.Desc(8, 64, 4, 32, 1, 2)]
    for d in unsupported:
        assert L.qfc_packed_size(ctypes.byref(d), ctypes.byref(out)) == 2
    assert L.qfc_packed_size(None, ctypes.byref(out)) == 1
    assert L.qfc_packed_size(ctypes.byref(binding.make_desc(8, 64, "w8c")), None) == 1


def test_argument_errors_before_any_launch(L):
    d = binding.make_desc(64, 64, "w8c")
    h = ctypes.c_void_p(0)
    a = ctypes.c_void_p(0x1000)   # never dereferenced: checks fail first
    odd = ctypes.c_void_p(0x1008)
    s = ctypes.c_void_p(0)
    assert L.qfc_pack_weights(ctypes.byref(d), None, a, a, 1 << 20, s, ctypes.byref(h)) == 1
    assert L.qfc_pack_weights(ctypes.byref(d), a, a, a, 1 << 20, s, None) == 1
    assert L.qfc_pack_weights(ctypes.byref(d), odd, a, a, 1 << 20, s, ctypes.byref(h)) == 4
    assert L.qfc_pack_weights(ctypes.byref(d), a, a, a, 16, s, ctypes.byref(h)) == 3
    assert h.value is None
    for fn, args in [(L.qfc_forward, (None, a, 1, a, s)), (L.qfc_forward_static, (None, a, 1, a, s)), (L.qfc_unpack_weights, (None, a, a, s)),
                     (L.qfc_bind_workspace, (None, a, 1024)), (L.qfc_forward_q8, (None, a, a, 1, a, s)),
                     (L.qfc_forward_acc_i32, (None, a, 1, a, s)), (L.qfc_embedding, (None, a, 1, a, s)),
                     (L.qfc_destroy, (None,))]:
        assert fn(*args) == 1
    out = ctypes.c_size_t(0)
    assert L.qfc_workspace_size(None, 1, ctypes.byref(out)) == 1
    assert L.qfc_quantize_activations(a, 0, 64, a, a, s) == 1
    assert L.qfc_quantize_activations(a, 4, 40, a, a, s) == 1
    assert L.qfc_quantize_activations(odd, 4, 64, a, a, s) == 4
    assert L.qfc_quantize_activations(None, 4, 64, a, a, s) == 1
    assert L.qfc_forward_batch(None, None, 1, None, 0, s) == 1
    assert L.qfc_forward_fused(None, a, 1, a, None, s) == 1
    # RMS normalization: argument checks come before any launch
    R = binding.RmsNorm
    A, ODD = 0x1000, 0x1008
    assert L.qfc_rmsnorm(None, 1, 64, s) == 1
    assert L.qfc_rmsnorm(ctypes.byref(R(A, None, A, 1e-5, 0.0, None, None, None, None)), 1, 64, s) == 1   # no output
    assert L.qfc_rmsnorm(ctypes.byref(R(A, None, A, 1e-5, 0.0, None, A, A, None)), 1, 64, s) == 1        # xq without sx
    assert L.qfc_rmsnorm(ctypes.byref(R(A, None, A, 1e-5, 0.0, None, A, None, None)), 1, 40, s) == 1      # K % 32
    assert L.qfc_rmsnorm(ctypes.byref(R(A, None, A, -1.0, 0.0, None, A, None, None)), 1, 64, s) == 1      # eps < 0
    assert L.qfc_rmsnorm(ctypes.byref(R(A, None, A, 1e-5, 0.0, None, A, None, None)), 1, 14368, s) == 2   # row too long
    assert L.qfc_rmsnorm(ctypes.byref(R(A, ODD, A, 1e-5, 0.0, None, A, None, None)), 1, 64, s) == 4
    assert L.qfc_rmsnorm(ctypes.byref(R(None, None, A, 1e-5, 0.0, None, A, None, None)), 1, 64, s) == 1
    # attention-side operators
    S8 = binding.AttnShape
    A = ctypes.c_void_p(0x1000)
    out = ctypes.c_size_t(0)
    assert L.qfc_attention_workspace_size(ctypes.byref(S8(1, 32, 8, 128, 4096)), 1, ctypes.byref(out)) == 0
    assert out.value == 8 * 64 * 4 * 130 * 4
    assert L.qfc_attention_workspace_size(ctypes.byref(S8(1, 32, 8, 96, 4096)), 1, ctypes.byref(out)) == 2    # head size
    assert L.qfc_attention_workspace_size(ctypes.byref(S8(1, 32, 8, 128, 4128)), 1, ctypes.byref(out)) == 1   # cache % 64
    assert L.qfc_attention_workspace_size(ctypes.byref(S8(1, 32, 6, 128, 4096)), 1, ctypes.byref(out)) == 1   # h_q % h_kv
    assert L.qfc_attention_workspace_size(ctypes.byref(S8(1, 32, 8, 128, 4096)), 5, ctypes.byref(out)) == 0   # prefill path
    assert out.value == 256
    sh = S8(1, 32, 8, 128, 4096)
    assert L.qfc_attention(A, A, A, 1, 0, ctypes.byref(sh), A, 1 << 30, A, s) == 1        # n_ctx < S
    assert L.qfc_attention(A, A, A, 1, 5000, ctypes.byref(sh), A, 1 << 30, A, s) == 1     # n_ctx > cache
    assert L.qfc_attention(A, A, A, 1, 100, ctypes.byref(sh), A, 1024, A, s) == 3         # workspace too small
    assert L.qfc_attention(A, A, ctypes.c_void_p(0x1008), 1, 100, ctypes.byref(sh), A, 1 << 30, A, s) == 4
    assert L.qfc_rope_qkv(A, 1, 4096, ctypes.byref(sh), 10000.0, A, A, A, s) == 1           # position past the cache
    assert L.qfc_rope_qkv(A, 1, 0, ctypes.byref(sh), 1.0, A, A, A, s) == 1                  # base must exceed 1
    assert L.qfc_rope_qkv(None, 1, 0, ctypes.byref(sh), 10000.0, A, A, A, s) == 1


def test_build_refuses_spills_in_kernels_with_hand_placed_loads():
    """The build parses the compiler's resource-usage remarks of the kernels whose operand loads are
    asynchronous assembly (a spilled destination register would be saved before its load lands)."""
    from paper_2505_00232_amd import build
    pre = "gemm_i8.hip:527:1: remark: "
    suf = " [-Rpass-analysis=kernel-resource-usage]"
    def remarks(name, scratch, vspill):
        return [pre + f"Function Name: {name}" + suf, pre + "    VGPRs: 220" + suf,
                pre + f"    ScratchSize [bytes/lane]: {scratch}" + suf, pre + "    SGPRs Spill: 0" + suf,
                pre + f"    VGPRs Spill: {vspill}" + suf]
    clean = remarks("_ZN3qfc17gemm_i8_dw_kernelILb1ELi8ELi4ELi2ELi0EEEv", 0, 0)
    other = remarks("_ZN3qfc14gemm_i8_kernelILi128ELi128EEEv", 76, 18)   # not one of the guarded kernels
    bad = remarks("_ZN3qfc17gemm_i8_dw_kernelILb0ELi4ELi2ELi4ELi0EEEv", 76, 18)
    frag = build.NO_SPILL["gemm_i8.hip"]
    assert build._spilling_kernels(clean + other, frag) == []
    assert build._spilling_kernels(clean + bad + other, frag) == ["_ZN3qfc17gemm_i8_dw_kernelILb0ELi4ELi2ELi4ELi0EEEv"]


def test_build_sees_changes_of_its_flags_and_headers(tmp_path, monkeypatch):
    """A library older than any source, public header or the build's own file is built again."""
    include = os.path.join(ROOT, "include")
    for changed in [build.__file__] + [os.path.join(include, f) for f in os.listdir(include)] + [os.path.join(build.CSRC, "attention_walk.h")]:
        real = os.path.getmtime
        newest = str(tmp_path / "lib")
        open(newest, "w").close()
        monkeypatch.setattr(build.os.path, "getmtime", lambda p: 3 if os.path.realpath(p) == os.path.realpath(changed) else 2 if p == newest else 1)
        stale = build._deps_newer(newest)
        monkeypatch.setattr(build.os.path, "getmtime", real)
        assert stale, changed


_IN_A_PROCESS = """import sys, types, warnings
{0}
from paper_2505_00232_amd import binding
with warnings.catch_warnings(record=True) as said:
    warnings.simplefilter("always")
    binding.lib()
assert {1}, (binding._fast, [str(w.message) for w in said])
assert binding.status_string(0) == "ok"
for call in (lambda h, x: binding.qfc_forward(h, x, x), lambda h, x: binding.qfc_forward_fused(h, x, x)):
    import ctypes, torch
    binding._dims[4096] = (64, 64)
    try:
        call(ctypes.c_void_p(4096), torch.zeros(2, 64, dtype=torch.float16))
    except ValueError as e:
        assert "CUDA tensor" in str(e)
    else:
        raise AssertionError("a host tensor was taken")
"""


@pytest.mark.parametrize("before,after", [
    ("", "binding._fast is not None and not said"),  # as it is built here
    ("sys.modules['paper_2505_00232_amd._marshal'] = None", "binding._fast is None and len(said) == 1"),  # missing, or the loader refuses it
    ("m = types.ModuleType('paper_2505_00232_amd._marshal'); m.built_for = 'Python 3.10, torch 1.0'; sys.modules[m.__name__] = m",
     "binding._fast is None and len(said) == 1 and 'torch 1.0' in str(said[0].message)"),  # built against another torch
    ("m = types.ModuleType('paper_2505_00232_amd._marshal'); sys.modules[m.__name__] = m", "binding._fast is None and len(said) == 1")])  # one that does not say
def test_binding_works_without_the_native_module(L, before, after):
    """_marshal only shortens the way of two calls: without it the library loads, and every call goes through ctypes."""
    r = subprocess.run([sys.executable, "-c", _IN_A_PROCESS.format(before, after)], cwd=ROOT, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]


def test_build_sees_another_torch_and_lives_without_the_native_module(tmp_path, monkeypatch):
    """The native module is built again for another torch, and one that cannot be built is no error, but leaves no old one behind."""
    build.build()
    assert not build._marshal_stale()
    monkeypatch.setattr(binding.torch, "__version__", "99.0")
    assert build._marshal_stale()
    so = tmp_path / "_marshal.so"
    so.write_text("old")
    monkeypatch.setattr(build, "MARSHAL", str(so))
    monkeypatch.setattr(build, "MARSHAL_FOR", str(tmp_path / "for"))
    monkeypatch.setattr(build, "CSRC", str(tmp_path))  # (no marshal.cpp there)
    with pytest.warns(RuntimeWarning, match="could not be built"):
        build._build_marshal()
    assert not so.exists()


def test_prefill_walk_copies_land_before_they_are_read_and_end_with_the_walk(tmp_path):
    """The order in which the prefill attention kernel issues its copies, waits and reads, run on the host for every
    instance's rings, 1 to 25 steps and any share of unmasked stages: no copy past the walk, every step
    copied once, no slot overwritten while it is read or read before it is filled, nothing in flight at the end."""
    exe = str(tmp_path / "attention_walk")
    subprocess.run(["g++", "-std=c++17", "-O1", "-w", "-D__host__=", "-D__device__=", "-D__forceinline__=inline", "-I", build.CSRC,
                    os.path.join(ROOT, "tests", "attention_walk.cpp"), "-o", exe], check=True)
    r = subprocess.run([exe], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout[-2000:]


def test_reads_of_lds_stay_behind_the_wait_for_copies(tmp_path):
    """A kernel that reads a slot of LDS, waits for the copies into it and reads it again: two reads in the compiled code, one on
    each side of the wait."""
    from paper_2505_00232_amd import build
    src, out = tmp_path / "wait.hip", tmp_path / "wait.s"
    src.write_text("""#include "qfc_internal.h"
__global__ void k(uint32_t *y) {
    __shared__ uint32_t lds[256];
    qfc::copy16_to_lds(y, threadIdx.x * 16, (uint32_t)(uintptr_t)(__attribute__((address_space(3))) void *)lds);
    const uint32_t before = lds[threadIdx.x];
    qfc::wait_copies<3>();
    y[threadIdx.x] = before - lds[threadIdx.x];
}
""")
    subprocess.run([build._hipcc(), *build.FLAGS, "-w", "-I", build.CSRC, "--cuda-device-only", "-S", str(src), "-o", str(out)], check=True)
    code = [l.strip() for l in out.read_text().splitlines()]
    waits = [i for i, l in enumerate(code) if l.startswith("s_waitcnt") and "vmcnt(3)" in l]
    reads = [i for i, l in enumerate(code) if l.startswith("ds_read")]
    assert len(waits) == 1 and len(reads) == 2, (waits, reads)
    assert reads[0] < waits[0] < reads[1]


def test_tiles_copy_no_line_over_and_over(tmp_path):
    """The token rows that the binary16 tiles copy, for 9 to 400 rows and every number of rows per tile: the rows there are from their own
    place, the rows past the last from rows there are, and none of a wavefront's copies of a half stage more than twice from the same
    row (with 16 and 8 rows that the others may take: three and five times)."""
    src, exe = tmp_path / "rows.cpp", str(tmp_path / "rows")
    src.write_text("""#include "tile_rows.h"
#include <cstdio>
#include <map>
int main() {
    for (int rows = 32; rows <= 128; rows += 32)
        for (int M = 9; M <= 400; ++M)
            for (int m0 = 0; m0 < M; m0 += rows)
                for (int wave = 0; wave < 4; ++wave) {
                    std::map<int, int> copies;
                    for (int i = 0; i < rows / 32; ++i)
                        for (int r = 0; r < 8; ++r) {
                            const int at = m0 + 32 * i + 8 * wave + r, row = m0 - qfc::rows_in_front(m0, rows) + qfc::source_row(i, wave, r, m0, M, rows);
                            const int most = M >= 32 ? 2 : 1 + rows / (M >= 16 ? 64 : 32);
                            if (row < 0 || row >= M || (at < M && row != at) || ++copies[row] > most)
                                return printf("rows %d M %d m0 %d wave %d row %d from %d, copy %d\\n", rows, M, m0, wave, at, row, copies[row]), 1;
                        }
                }
    return 0;
}
""")
    subprocess.run(["g++", "-std=c++17", "-O1", "-D__host__=", "-D__device__=", "-D__forceinline__=inline", "-I", build.CSRC, str(src), "-o", exe], check=True)
    r = subprocess.run([exe], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout[-2000:]


def test_tile_order_covers_every_tile_once(tmp_path):
    """The walk over the tiles of a product: every tile once, for grids of one tile to several bands in both directions, bands of any
    width and any remainder over the XCDs; an XCD's neighbours stay within one band, or two where its share crosses over; and the walk that is chosen has equal
    bands, the last at most as many tiles narrower as there are others."""
    src, exe = tmp_path / "order.cpp", str(tmp_path / "order")
    src.write_text("""#include "tile_order.h"
#include <cstdio>
#include <vector>
int main() {
    for (int n = 1; n <= 40; ++n)
        for (int m = 1; m <= 40; ++m) {
            std::vector<qfc::TileWalk> walks = {{0, qfc::kBand}, {1, qfc::kBand}, {0, m}, {1, n}, {0, 5}, {1, 5}};
            for (int K : {512, 4096, 8192, 1000000})
                for (int i8 = 0; i8 < 2; ++i8) {
                    const qfc::TileWalk w = qfc::tile_walk(n, m, K, i8, 256.0f, 128.0f);
                    const int inner = w.by_tokens ? n : m, bands = (inner + w.band - 1) / w.band, last = inner - (bands - 1) * w.band;
                    if (w.band < 1 || w.band > inner || last < 1 || w.band - last >= bands + (bands == 1)) return printf("%d x %d: bands of %d, last %d\\n", n, m, w.band, last), 1;
                    walks.push_back(w);
                    walks.push_back(qfc::fewest_bytes_walk(n, m, 64.0f, 128.0f, false));
                }
            for (const qfc::TileWalk &walk : walks) {
                std::vector<int> seen(n * m, 0);
                for (int b = 0; b < n * m; ++b) {
                    int nt = -1, mt = -1;
                    qfc::xcd_tile(b, n, m, walk, nt, mt);
                    if (nt < 0 || nt >= n || mt < 0 || mt >= m || seen[nt * m + mt]++) return printf("%d x %d by_tokens %d band %d: %d -> %d %d\\n", n, m, walk.by_tokens, walk.band, b, nt, mt), 1;
                    if (b >= 8) {
                        int n0, m0;
                        qfc::xcd_tile(b - 8, n, m, walk, n0, m0);
                        const int band = (walk.by_tokens ? nt : mt) / walk.band - (walk.by_tokens ? n0 : m0) / walk.band;
                        if (band < 0 || band > 1) return printf("%d x %d by_tokens %d: band %d\\n", n, m, walk.by_tokens, band), 1;
                    }
                }
            }
        }
    return 0;
}
""")
    subprocess.run(["g++", "-std=c++17", "-O1", "-D__host__=", "-D__device__=", "-D__forceinline__=inline", "-I", build.CSRC, str(src), "-o", exe], check=True)
    r = subprocess.run([exe], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout[-2000:]


# channel tiles, token tiles, K, int8 activations, bytes of a channel tile and of a token tile per k: by tokens, tiles of a band
ORDERS = [
    # one band of channel tiles and many token tiles: int8 activations walk by tokens from twice (K up to 4096) or three times as many on
    (9, 18, 4096, 1, 256, 128, 1, 9), (9, 17, 4096, 1, 256, 128, 0, 9), (9, 32, 9216, 1, 256, 128, 1, 9), (9, 26, 9216, 1, 256, 128, 0, 9), (9, 32, 4096, 0, 256, 256, 0, 8),
    # equal bands: nine token tiles are one, twelve are two, thirteen seven and six
    (15, 9, 8448, 1, 128, 128, 0, 9), (20, 12, 4096, 1, 256, 128, 0, 6), (20, 13, 4096, 1, 256, 128, 0, 7),
    # more tiles than an XCD has in flight, several bands in both directions: by tokens, unless the weights are too many for the memory-side cache
    (112, 32, 4096, 1, 256, 128, 1, 8), (112, 47, 4096, 0, 128, 256, 1, 8), (133, 42, 13568, 1, 256, 128, 0, 42), (112, 8, 4096, 1, 256, 128, 0, 8),
    # without bands (K 0)
    (13, 33, 0, 1, 64, 128, 1, 13), (33, 13, 0, 1, 64, 128, 0, 13), (16, 17, 0, 1, 128, 64, 0, 17),
    # tiles that stage both operands (K negative): bands above 1024 of them
    (23, 32, -4000, 0, 72, 256, 1, 23), (32, 32, -4000, 0, 72, 256, 1, 32), (32, 33, -4000, 0, 72, 256, 1, 8), (13, 33, -1152, 1, 64, 128, 1, 13),
]


def test_tile_order_is_chosen_by_size(tmp_path):
    """In which order and in bands of how many tiles a product walks, on both sides of the rule's lines (times beside it); and the walk without bands."""
    src, exe = tmp_path / "walk.cpp", str(tmp_path / "walk")
    src.write_text("""#include "tile_order.h"
#include <cstdio>
int main() {
    for (int n, m, K, i8, w, x; scanf("%d %d %d %d %d %d", &n, &m, &K, &i8, &w, &x) == 6;) {
        const qfc::TileWalk walk = K == 0 ? qfc::fewest_bytes_walk(n, m, (float)w, (float)x, false) : K < 0 ? qfc::staged_tile_walk(n, m, -K, i8 != 0, (float)w, (float)x)
                                                                                                                          : qfc::tile_walk(n, m, K, i8 != 0, (float)w, (float)x);
        printf("%d %d\\n", walk.by_tokens, walk.band);
    }
}
""")
    subprocess.run(["g++", "-std=c++17", "-O1", "-D__host__=", "-D__device__=", "-D__forceinline__=inline", "-I", build.CSRC, str(src), "-o", exe], check=True)
    r = subprocess.run([exe], input="\n".join(" ".join(map(str, o[:6])) for o in ORDERS), capture_output=True, text=True, check=True)
    assert [(*o[:6], *map(int, l.split())) for o, l in zip(ORDERS, r.stdout.splitlines())] == ORDERS


def test_int8_tiles_wait_for_what_they_read(tmp_path):
    """The operations that a wavefront of the direct-weights int8 tiles issues, for every instance in gemm_i8.hip and 2 to 24 stages: where it
    goes on to read, even if loads, copies and touches of the weights each complete in order but in no order among them, no
    operation that the stage needs can be among as many as may be outstanding."""
    text = open(os.path.join(build.CSRC, "gemm_i8.hip")).read()
    forms = re.findall(r"launch_dw<(true|false), (\d+), (\d+), (\d+), (\d+), \d+, (true|false), OUT_MODE>\(a, st\)", text)
    assert len(forms) == text.count("launch_dw<") >= 9
    src, exe = tmp_path / "waits.cpp", str(tmp_path / "waits")
    src.write_text("""#include "tile_waits.h"
#include <cstdio>
#include <vector>
enum Kind { kLoad, kCopy, kTouch };
struct Op { Kind kind; int stage; };
int main() {
    for (int w4, NS, PW, TM, CG, touch; scanf("%d %d %d %d %d %d", &w4, &NS, &PW, &TM, &CG, &touch) == 6;) {
        const int copies = 4 * TM / CG, loads = w4 ? 4 : 8;
        const bool pipe = !w4 && TM == 2 && !touch;
        const qfc::DwWaits waits = qfc::dw_waits(copies, loads, NS, PW, pipe);
        for (int KT = 2; KT <= 24; KT += 2) {
            std::vector<Op> issued;
            auto issue = [&](Kind kind, int stage, int n) { while (n-- > 0) issued.push_back({kind, stage}); };
            auto safe = [&](Kind kind, int stage, int allowed) {  // the fewest outstanding with any of the stage's operations among them
                for (size_t i = 0; i < issued.size(); ++i) {
                    if (issued[i].kind != kind || issued[i].stage != stage) continue;
                    int outstanding = 0;
                    for (size_t j = i; j < issued.size(); ++j) outstanding += issued[j].kind == kind;
                    if (outstanding <= allowed) return printf("w4 %d NS %d PW %d TM %d CG %d touch %d, %d stages: kind %d of stage %d, %d of %d\\n", w4, NS, PW, TM, CG, touch, KT, kind, stage, outstanding, allowed), false;
                }
                return true;
            };
            for (int p = 0; p < PW; ++p) issue(kLoad, p, loads);
            for (int p = 0; p < NS - 1; ++p) issue(kCopy, p, copies), issue(kTouch, PW + p, touch);
            if (pipe && !safe(kCopy, 0, waits.first)) return 1;
            for (int kt = 0; kt < KT; ++kt) {
                if (!safe(kLoad, kt, waits.allowed) || !safe(kCopy, pipe ? kt + 1 : kt, waits.allowed)) return 1;
                issue(kCopy, kt + NS - 1, copies), issue(kTouch, kt + NS - 1 + PW, touch);
                issue(kLoad, kt + PW, loads);
            }
        }
    }
    return 0;
}
""")
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", build.CSRC, str(src), "-o", exe], check=True)
    asked = "\n".join(" ".join({"true": "1", "false": "0"}.get(v, v) for v in f) for f in forms)
    r = subprocess.run([exe], input=asked, capture_output=True, text=True)
    assert r.returncode == 0, r.stdout[-2000:]


# What the dispatch chooses on 256 compute units.  Binary16 activations: format (0 int8, 1 int4 in groups, 2 int4), channels, K, token rows,
# rows left to the token-row kernels in a second launch (-1: they take them all)
CHOICES = [
    # K of less than 256: one launch (us, two / one: 8192 x 128 1030 rows 10.9 / 8.5, 10807 x 128 706 rows 20.0 / 7.8, int8 10501 x 64 1001 rows 19.4 / 9.4)
    (1, 8192, 128, 1030, 0), (2, 8192, 128, 1030, 0), (2, 10807, 128, 706, 0), (0, 10501, 64, 1001, 0), (0, 8192, 192, 1030, 0),
    # K of 512 and less, few tiles, and the token-row kernels half a microsecond faster or more; up to 16 rows
    (0, 1404, 192, 73, -1), (2, 311, 256, 442, -1), (1, 3527, 256, 69, -1), (0, 9668, 256, 24, -1), (0, 345, 256, 146, -1), (0, 34177, 512, 12, -1), (1, 80000, 1024, 9, -1),
    # more rows and many channels: the tiles
    (2, 28000, 512, 20, 0), (1, 128256, 4096, 32, 0), (0, 29780, 512, 28, 0),
    # two launches where those are the faster ones
    (2, 4096, 4096, 2060, 12), (1, 2304, 9216, 3700, 116), (1, 3072, 1536, 2698, 10), (0, 2048, 1536, 4100, 4),
]
# int8 activations and weights: channels, K, token rows, whether the workgroups stay and walk over row tiles
STREAMS = [(128256, 4096, 24, 1), (65536, 8192, 9, 1), (31104, 8192, 24, 1), (152064, 512, 24, 1), (140000, 512, 9, 1), (250000, 512, 24, 1), (65535, 992, 17, 1), (57344, 4096, 9, 1), (99936, 4096, 24, 1), (128256, 4096, 9, 1),
           # not: a last round of few workgroups with K of 8192; K of 512 and 1024, many channels and up to 16 rows, or rows of single values
           (33000, 8192, 16, 0), (50304, 8192, 24, 0), (28672, 4096, 20, 0), (250000, 512, 9, 0), (200000, 1024, 16, 0), (131070, 512, 32, 0), (200001, 1024, 32, 0),
           (164748, 992, 10, 0), (99936, 4096, 9, 0), (131758, 4096, 10, 0), (202048, 2048, 24, 0), (128256, 4096, 33, 0)]

# int8 activations, rows past the token-row kernels' own: format, channels, K, token rows, the form of the tiles (0: the token-row kernels)
INT8_TILES = [
    # int8 weights: 256 x 128, 256 x 64 and, K in two parts, 128 x 128 and 128 x 64
    (0, 4096, 14336, 512, 14), (0, 4096, 14336, 1024, 13), (0, 4096, 14336, 1100, 10), (0, 4096, 14336, 2048, 10), (0, 6144, 4096, 1024, 10), (0, 2112, 6144, 505, 14),
    (0, 1600, 2048, 2026, 12), (0, 30336, 12544, 96, 12), (0, 28672, 4096, 66, 12), (0, 28672, 4096, 129, 10), (0, 4096, 768, 512, 14), (0, 4096, 256, 300, 12),
    # int4 weights: 256 x 128, 256 x 64, 128 x 64 with K in two and in four parts
    (2, 28672, 4096, 1024, 21), (2, 9008, 1024, 600, 21), (2, 4096, 4096, 512, 24), (2, 2304, 9216, 814, 25), (2, 4096, 512, 300, 24),
    # the line between the tiles and the token-row kernels: rows, and rows that are stored value by value
    (0, 4096, 14336, 191, 0), (0, 4096, 9216, 214, 0), (0, 4096, 9216, 300, 14), (0, 6144, 4096, 150, 0), (0, 6144, 4096, 240, 14), (2, 4096, 14336, 100, 0), (2, 4096, 14336, 300, 25),
    (2, 2304, 9216, 300, 0), (2, 2304, 9216, 500, 25), (0, 9001, 1024, 600, 0), (0, 9000, 1024, 600, 10), (0, 4635, 1280, 420, 0), (0, 4640, 1280, 420, 12), (2, 8482, 1024, 230, 0),
]


def test_choice_of_kernels(tmp_path):
    """The dispatch's own functions, compiled for the host, on both sides of its lines (times of both beside the rules)."""
    src, obj, exe = tmp_path / "choice.hip", str(tmp_path / "choice.o"), str(tmp_path / "choice")
    src.write_text("""#include "gemm_skinny.hip"
#include <cstdio>
int main() {
    for (int kind, fmt, N, K, M; scanf("%d %d %d %d %d", &kind, &fmt, &N, &K, &M) == 5;) {
        const qfc::Geometry g = qfc::make_geometry(N, K, fmt);
        if (kind == 0)
            printf("%d\\n", qfc::skinny_product(g, M, false, false, 256) ? -1 : qfc::skinny_tail_rows(g, M, false, 256));
        else if (kind == 1)
            printf("%d\\n", (int)qfc::stream_takes(qfc::make_args(g, nullptr, nullptr, nullptr, M, nullptr, nullptr, -1), 256));
        else {
            int form;
            qfc::int8_tile_us(g, M, N % 8 == 0, 256, &form);
            printf("%d\\n", qfc::skinny_product(g, M, true, false, 256) ? 0 : form);
        }
    }
}
""")
    binding.lib()
    where = os.path.dirname(build.LIB)
    subprocess.run([build._hipcc(), "-std=c++17", "-w", "-O1", "-fPIC", "--offload-arch=gfx950", "--cuda-host-only", "-I", build.CSRC, "-c", str(src), "-o", obj], check=True)
    # (no device code: the kernels' images are never looked up)
    subprocess.run([build._hipcc(), obj, "-o", exe, "-Wl,--unresolved-symbols=ignore-all", "-L", where, "-lqfc", "-Wl,-rpath," + where], check=True)
    asked = [(0, *c[:4]) for c in CHOICES] + [(1, 0, *s[:3]) for s in STREAMS] + [(2, *t[:4]) for t in INT8_TILES]
    r = subprocess.run([exe], input="\n".join(" ".join(map(str, c)) for c in asked), capture_output=True, text=True, check=True)
    got = [int(v) for v in r.stdout.split()]
    assert got[:len(CHOICES)] == [c[4] for c in CHOICES]
    assert got[len(CHOICES):len(CHOICES) + len(STREAMS)] == [s[3] for s in STREAMS]
    assert got[len(CHOICES) + len(STREAMS):] == [t[4] for t in INT8_TILES]


# KV heads, query rows per head, head size, positions: workgroups per KV head on 256 compute units
WALKS = [(8, 4, 128, 1280, 20), (56, 4, 128, 3000, 4), (256, 4, 128, 3000, 1), (20, 2, 256, 9000, 12),
         # more KV heads than compute units: four walks from 14 steps and positions x idle share of the last round = heads x (1.8 + 0.15 rows) on, a last
         # round of 35 % at most
         (257, 1, 128, 833, 4), (257, 1, 128, 832, 1), (257, 16, 64, 1083, 1), (257, 16, 64, 1084, 4), (257, 16, 256, 1083, 1), (257, 16, 256, 1084, 4), (345, 1, 128, 3000, 4), (346, 1, 128, 3000, 1),
         (512, 1, 128, 9000, 1), (520, 1, 128, 1500, 4), (520, 16, 128, 1500, 1), (2064, 1, 64, 4294, 4), (2064, 1, 64, 4293, 1),
         # short walks and many heads (us, one / four: 4112 heads of 256, 448 positions, 16 rows 389 / 607; 264 of 256, 448, 8 rows 12 % slower)
         (4112, 16, 256, 448, 1), (4112, 1, 256, 448, 1), (264, 8, 256, 448, 1), (2561, 1, 128, 1500, 1)]


def test_decode_attention_walks():
    """Into how many walks the decode attention of a KV head is cut, on both sides of the rule's lines (times beside it)."""
    binding.lib()
    splits = ctypes.CDLL(binding.LIB_PATH)._ZN3qfc11attn_splitsEiiiii
    got = [(*w[:4], splits(*w[:4], 256)) for w in WALKS]
    assert got == WALKS


# tokens, heads that are rotated, head size: tokens per workgroup of the rotary embedding of many tokens
ROTATIONS = [(816, 12, 128, 1), (1939, 10, 64, 3), (1216, 3, 128, 2), (1023, 3, 128, 1), (4793, 2, 64, 8), (1024, 40, 128, 1), (2047, 40, 128, 1), (2048, 40, 128, 2), (6000, 40, 128, 4),
             (6000, 12, 256, 2), (128, 8, 256, 1), (1100, 6, 64, 2), (100000, 3, 64, 8)]


def test_rope_tokens_per_workgroup():
    """On both sides of the rule's lines (times beside it)."""
    binding.lib()
    tokens = ctypes.CDLL(binding.LIB_PATH)._ZN3qfc11rope_tokensElii
    assert [(*r[:3], tokens(ctypes.c_long(r[0]), *r[1:3])) for r in ROTATIONS] == ROTATIONS
