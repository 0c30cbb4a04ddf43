"""Host-side checks of the C ABI (no GPU): the library loads, exports every declared symbol, and
refuses bad arguments before anything is launched."""
import ctypes
import os
import re
import shutil
import subprocess
import sys

import pytest

import paper_2412_16481_amd as f3d

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def declared_symbols():
    text = open(os.path.join(ROOT, "include", "flash3d.h")).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    names = set(re.findall(r"\b(f3d_[a-z0-9_]+)\s*\(", text))
    names.discard("f3d_psh_bucketize_simple")          # static inline wrapper in the header
    return sorted(names)


def test_library_exports_every_declared_symbol():
    L = f3d.lib()
    names = declared_symbols()
    assert set(names) == set(f3d.EXPORTS)
    for name in names:
        assert getattr(L, name) is not None
    assert f3d.version() >= 1


def test_microbenchmark_library_is_built_and_refuses_bad_arguments_on_the_host():
    # the measurement aid of bench.py --ceilings: built by the same build step, one entry point, checked before any GPU call
    mb = ctypes.CDLL(os.path.join(ROOT, "paper_2412_16481_amd", "libf3d_microbench.so"))
    mb.f3d_mb_run.argtypes = [ctypes.c_int, ctypes.c_int, ctypes.POINTER(ctypes.c_float), ctypes.POINTER(ctypes.c_double)]
    ms, work = ctypes.c_float(0), ctypes.c_double(0)
    assert mb.f3d_mb_run(8, 4, ctypes.byref(ms), ctypes.byref(work)) != 0
    assert mb.f3d_mb_run(0, 0, ctypes.byref(ms), ctypes.byref(work)) != 0
    assert mb.f3d_mb_run(0, 9, ctypes.byref(ms), ctypes.byref(work)) != 0
    assert mb.f3d_mb_run(0, 4, None, ctypes.byref(work)) != 0


def test_every_load_into_lds_waits_for_the_write_of_m0(tmp_path):
    # a load into LDS takes its address from M0, which needs one wait state behind a scalar write of it; the compiler does
    # not insert that inside assembly statements, so the built code is looked through
    objdump = "/opt/rocm/llvm/bin/llvm-objdump"
    if not os.path.exists(objdump):
        pytest.skip("no llvm-objdump here")
    shutil.copy(f3d.LIB_PATH, tmp_path / "lib.so")
    subprocess.run([objdump, "--offloading", "lib.so"], cwd=tmp_path, check=True, capture_output=True)
    loads = 0
    for part in tmp_path.glob("lib.so.*gfx950*"):
        text = subprocess.run([objdump, "-d", part.name], cwd=tmp_path, check=True, capture_output=True, text=True).stdout
        before = ""
        for line in (x.split("//")[0].strip() for x in text.splitlines()):
            if re.match(r"(global|scratch)_load_lds_|buffer_load_.*\blds\b", line):
                loads += 1
                assert not re.match(r"s_\w+ m0\b", before), f"{part.name}: {before}; {line}"
            before = line or before
    assert loads > 0


RECORDING_RUNTIME = r"""
// stands in for the HIP runtime on a machine without a GPU: says what LDS a kernel is allowed and what every launch asks for
#include <stddef.h>
#include <stdio.h>
typedef struct { unsigned x, y, z; } dim3;
static size_t lds;
int hipFuncSetAttribute(const void* f, int attr, int value) { fprintf(stderr, "allow %p %d %d\n", f, attr, value); return 0; }
int hipLaunchKernel(const void* f, dim3 g, dim3 b, void** args, size_t bytes, void* s) { fprintf(stderr, "launch %p %zu\n", f, bytes); return 0; }
int __hipPushCallConfiguration(dim3 g, dim3 b, size_t bytes, void* s) { lds = bytes; return 0; }
int __hipPopCallConfiguration(dim3* g, dim3* b, size_t* bytes, void** s)
{
    const dim3 one = {1, 1, 1};
    *g = one; *b = one; *bytes = lds; *s = 0;
    return 0;
}
int hipGetDevice(int* d) { *d = 0; return 0; }
int hipDeviceGetAttribute(int* v, int attr, int d) { *v = 256; return 0; }
int hipGetLastError(void) { return 0; }
void** __hipRegisterFatBinary(const void* data) { static void* h; return &h; }
void __hipRegisterFunction(void** m, const void* f, char* d, const char* n, unsigned l, void* t, void* b, void* bd, void* gd, int* w) {}
void __hipRegisterVar(void** m, void* v, char* h, char* d, int e, size_t size, int c, int g) {}
void __hipUnregisterFatBinary(void** m) {}
"""

CALLS_OF_MANY_SIZES = """
import ctypes, sys
from ctypes import byref, c_float, c_int32, c_int64, c_size_t, c_void_p
ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
import paper_2412_16481_amd as f3d
L = ctypes.CDLL(f3d.LIB_PATH)
at, big = c_void_p(0x10000), c_size_t(1 << 40)     # never followed: nothing is launched
def bucketize(n, scans, most, cap, hash="zorder_div", schedule="auto"):
    p = f3d.make_params(0.05, cap, hash=hash, max_scan_points=most, schedule=schedule)
    return L.f3d_psh_bucketize(at, None, c_int64(n), scans, byref(p), at, None, at, at, None, at, big, None)
def pool(n, tile, rho):
    return L.f3d_inbucket_pool(at, None, at, None, c_int64(n), 1, 8, tile, rho, c_float(0.1), 3, 0, at, None, None, at, at, big, None)
def linear(c_in, c_out):
    return L.f3d_ln_linear(at, None, None, None, c_float(0), at, None, None, c_int64(100), c_in, c_out, (c_void_p * 1)(0x10000), 1, None, None)
rc = []
for n in (3000, 3000000):
    for tile in (66, 256, 640, 1024):
        rc += [pool(n, tile, rho) for rho in (1, 2, 4)]
for hash in ("xor_mod", "xor_div", "zorder_mod", "zorder_div"):
    for scans in (60, 600):
        rc += [bucketize(scans * most, scans, most, cap, hash, "scans") for most in (900, 5000, 50000) for cap in (256, 1024) if 4 * most <= 1024 * cap]
rc += [bucketize(n, 1, n, cap) for n in (500, 3000, 5000, 8000) for cap in (64, 1024)]
rc += [bucketize(n, 1, n, cap, schedule="steps") for n in (3000, 30000, 200000) for cap in (64, 256, 1024) if 4 * n <= 2048 * cap and n * n // cap < 1 << 25]
rc += [bucketize(n, 1, n, cap, schedule="general") for n in (30000, 500000) for cap in (256, 1024)]
rc += [linear(c_in, c_out) for c_in in (64, 128, 256) for c_out in (64, 3648, 4096)]
print("codes", *rc)
"""


def test_lds_allowed_to_a_kernel_is_the_same_in_every_call(tmp_path):
    """How much dynamic LDS a kernel may be launched with is a setting of the kernel, shared by all threads of the process. If a call
    set it to what it needs itself, a smaller call of another thread could lower it between that setting and the launch."""
    cc = shutil.which("gcc") or shutil.which("cc")
    if cc is None:
        pytest.skip("no C compiler here")
    (tmp_path / "hip.c").write_text(RECORDING_RUNTIME)
    (tmp_path / "calls.py").write_text(CALLS_OF_MANY_SIZES)
    subprocess.run([cc, "-shared", "-fPIC", "-w", "-fno-builtin", "-o", tmp_path / "hip.so", tmp_path / "hip.c"], check=True)
    run = subprocess.run([sys.executable, tmp_path / "calls.py", tmp_path / "hip.so"], cwd=ROOT, env={**os.environ, "PYTHONPATH": ROOT},
                         capture_output=True, text=True)
    assert run.returncode == 0, run.stderr
    allowed, launches = {}, 0
    assert set(run.stdout.split()) == {"codes", "0"}
    for word in (line.split() for line in run.stderr.splitlines()):
        if word[0] == "allow":
            assert allowed.setdefault(word[1], word[2:]) == word[2:], "set to two values"
        elif word[0] == "launch":
            assert int(word[2]) <= int(allowed.get(word[1], [0, 65536])[1])
            launches += 1
    assert len(allowed) >= 18 and launches > 100     # pooling 2, one workgroup per scan 8, small scans 3, a launch per step 2, general 1, linear 2


def test_params_default_and_sizes():
    p = f3d.make_params(0.02, 1024)
    assert p.struct_size == ctypes.sizeof(f3d.f3d_params)
    assert (p.scope_buckets, p.hash, p.n_probes, p.div, p.probe_step) == (4, 3, 6, 0, 0)
    assert f3d.max_buckets(200_000, 1, p) == 200_000 // 256 + 1
    assert f3d.workspace_bytes(200_000, 1, p) > 200_000 * 8
    assert f3d.workspace_bytes(0, 1, p) > 0


@pytest.mark.parametrize("kw,code", [
    (dict(voxel_size=0.0), f3d.ERR_INVALID_ARG),
    (dict(voxel_size=-1.0), f3d.ERR_INVALID_ARG),
    (dict(voxel_size=float("nan")), f3d.ERR_INVALID_ARG),
    (dict(bucket_cap=1000), f3d.ERR_INVALID_ARG),            # not a multiple of 16 * scope_buckets
    (dict(scope_buckets=0), f3d.ERR_INVALID_ARG),
    (dict(scope_buckets=32, bucket_cap=1024), f3d.ERR_UNSUPPORTED),
    (dict(hash=7), f3d.ERR_INVALID_ARG),
    (dict(n_probes=7), f3d.ERR_INVALID_ARG),
    (dict(n_probes=-1), f3d.ERR_INVALID_ARG),
    (dict(div=-1), f3d.ERR_INVALID_ARG),
    (dict(n=-1), f3d.ERR_INVALID_ARG),
    (dict(n_scans=0), f3d.ERR_INVALID_ARG),
    (dict(n=10_000_000, bucket_cap=64), f3d.ERR_UNSUPPORTED),  # one scan would own > 8192 buckets
    (dict(struct_size=4), f3d.ERR_INVALID_ARG),
    (dict(order=2), f3d.ERR_INVALID_ARG),
    (dict(order=-1), f3d.ERR_INVALID_ARG),
    (dict(probe_mode=3), f3d.ERR_INVALID_ARG),
    (dict(probe_mode=-1), f3d.ERR_INVALID_ARG),
])
def test_workspace_query_refuses_bad_parameters(kw, code):
    kw = dict(kw)
    n = kw.pop("n", 1000)
    n_scans = kw.pop("n_scans", 1)
    struct_size = kw.pop("struct_size", None)
    base = dict(voxel_size=0.02, bucket_cap=1024)
    base.update(kw)
    p = f3d.make_params(**base)
    if struct_size is not None:
        p.struct_size = struct_size
    out = ctypes.c_size_t(0)
    assert f3d.lib().f3d_workspace_bytes(n, n_scans, ctypes.byref(p), ctypes.byref(out)) == code


def test_rebalancing_variants_in_the_parameter_block():
    p = f3d.make_params(0.02, 1024)
    assert (p.order, p.probe_mode, p.probe_seed) == (0, 0, 0) and list(p.probe_table) == [0] * 18
    q = f3d.make_params(0.02, 1024, order="canonical", probe_mode="table", probe_seed=-1, probe_table=[[1, -2, 3], [4, 5, -6]])
    assert (q.order, q.probe_mode, q.probe_seed) == (1, 1, 0xFFFFFFFF)
    assert list(q.probe_table)[:6] == [1, -2, 3, 4, 5, -6]
    with pytest.raises(ValueError):
        f3d.make_params(0.02, 1024, probe_table=[[0, 0, 0]] * 7)
    # the canonical order sorts the points first and needs room for keys, indices and the sorted copy
    assert f3d.workspace_bytes(200_000, 1, q) > f3d.workspace_bytes(200_000, 1, p) + 200_000 * 48


def test_half_precision_attention_refuses_what_the_bfloat16_entry_refuses():
    L = f3d.lib()
    fake = 0x10000
    base = [fake, fake, fake, None, fake, fake, 100, 1, 10, 1024, 4, 0, 2, 2, 4, 16, 0.0, fake, None, None, None]
    def call(entry, changes):
        a = list(base)
        for k, v in changes.items():
            a[k] = v
        return entry(*a)
    for entry in (L.f3d_bucket_swin_attn, L.f3d_bucket_swin_attn_f16):
        assert call(entry, {15: 24}) == f3d.ERR_UNSUPPORTED        # head_dim
        assert call(entry, {0: None}) == f3d.ERR_INVALID_ARG       # q
        assert call(entry, {17: None}) == f3d.ERR_INVALID_ARG      # out
        assert call(entry, {17: fake + 8}) == f3d.ERR_BAD_ALIGNMENT
        assert call(entry, {11: 3}) == f3d.ERR_INVALID_ARG         # mode
        assert call(entry, {6: 0}) == 0                            # an empty input is not an error and launches nothing


def test_max_scan_points_lifts_the_bucket_limit():
    p = f3d.make_params(0.02, 64, max_scan_points=100_000)
    assert f3d.workspace_bytes(10_000_000, 200, p) > 0


@pytest.mark.parametrize("order", ["index", "canonical"])
@pytest.mark.parametrize("cap", [64, 192, 1024, 2048])
def test_workspace_never_shrinks_as_the_batch_grows(cap, order):
    """A program that allocates once for its largest batch reuses the buffer for every smaller one. The sizes walk over the limits
    of the chunks of 1024 points: 92 160 to 262 144 points, depending on buckets, scans and the largest scan. (From 48 scans on the
    lists of the path with one workgroup per scan come and go with n; those are not looked at here.)"""
    def size(n, n_scans, most):
        return f3d.workspace_bytes(n, n_scans, f3d.make_params(0.05, cap, 4, max_scan_points=most, order=order))

    near = [e + d for e in (92160, 131072, 185344, 215040, 255000, 261120, 262144) for d in range(-3, 4)]
    grow = sorted(set(near) | set(range(1, 300000, 1021)))
    for n_scans in (1, 2, 8, 47):
        for most in (0, 20000):
            sizes = [size(n, n_scans, most) for n in grow if (min(n, most or n) + cap // 4 - 1) // (cap // 4) <= 8192]
            assert sizes == sorted(sizes), (n_scans, most)
    for n in (1000, 150000, 250000):
        sizes = [size(n, n_scans, 5000) for n_scans in range(1, 513)]
        assert sizes == sorted(sizes), n
        sizes = [size(n, 8, most) for most in sorted(set(m for m in near if m <= n) | set(range(1000, n, 1021))) if 4 * most <= 8192 * cap]
        assert sizes == sorted(sizes), n


def test_bucketize_refuses_null_and_misaligned_pointers_on_the_host():
    L = f3d.lib()
    p = f3d.make_params(0.02, 1024)
    fake = 0x10000  # never dereferenced: the checks fail first
    args = lambda **o: [o.get("coords", fake), None, 100, 1, ctypes.byref(p), o.get("perm", fake), None,
                        o.get("offsets", fake), o.get("sbs", fake), None, o.get("ws", fake), o.get("wsb", 1 << 30), None]
    assert L.f3d_psh_bucketize(*args(coords=None)) == f3d.ERR_INVALID_ARG
    assert L.f3d_psh_bucketize(*args(perm=None)) == f3d.ERR_INVALID_ARG
    assert L.f3d_psh_bucketize(*args(offsets=None)) == f3d.ERR_INVALID_ARG
    assert L.f3d_psh_bucketize(*args(ws=None)) == f3d.ERR_INVALID_ARG
    assert L.f3d_psh_bucketize(*args(coords=fake + 2)) == f3d.ERR_BAD_ALIGNMENT
    assert L.f3d_psh_bucketize(*args(ws=fake + 64)) == f3d.ERR_BAD_ALIGNMENT
    assert L.f3d_psh_bucketize(*args(wsb=16)) == f3d.ERR_WORKSPACE_TOO_SMALL


def test_attention_refuses_bad_arguments_on_the_host():
    L = f3d.lib()
    fake = 0x10000
    def call(**o):
        return L.f3d_bucket_swin_attn(o.get("q", fake), fake, fake, None, o.get("offsets", fake), fake, o.get("n", 100), 1, 10,
                                      o.get("cap", 1024), o.get("m", 4), o.get("mode", 0), o.get("shift", 2),
                                      o.get("stride", 2), o.get("heads", 4), o.get("d", 16), o.get("scale", 0.0), fake, o.get("out_perm"), o.get("lse"), None)
    assert call(d=24) == f3d.ERR_UNSUPPORTED
    assert call(d=64) == f3d.ERR_UNSUPPORTED
    assert call(mode=3) == f3d.ERR_INVALID_ARG
    assert call(mode=1, shift=0) == f3d.ERR_INVALID_ARG
    assert call(mode=1, shift=4) == f3d.ERR_INVALID_ARG
    assert call(mode=2, stride=0) == f3d.ERR_INVALID_ARG
    assert call(cap=1000) == f3d.ERR_INVALID_ARG
    assert call(heads=0) == f3d.ERR_INVALID_ARG
    assert call(scale=-1.0) == f3d.ERR_INVALID_ARG
    assert call(q=None) == f3d.ERR_INVALID_ARG
    assert call(out_perm=fake + 2) == f3d.ERR_BAD_ALIGNMENT
    assert call(lse=fake + 1) == f3d.ERR_BAD_ALIGNMENT
    assert call(q=fake + 2) == f3d.ERR_BAD_ALIGNMENT
    assert call(offsets=None) == f3d.ERR_INVALID_ARG
    assert call(n=-5) == f3d.ERR_INVALID_ARG
    assert call(n=0) == f3d.F3D_OK                      # nothing to do, nothing launched


def test_unpermute_refuses_bad_arguments_on_the_host():
    L = f3d.lib()
    fake = 0x10000
    assert L.f3d_unpermute(fake, fake, 10, 0, fake + 4096, None) == f3d.ERR_INVALID_ARG
    assert L.f3d_unpermute(fake, fake, 10, 6, fake + 4096, None) == f3d.ERR_INVALID_ARG
    assert L.f3d_unpermute(fake, fake, 10, 128, fake, None) == f3d.ERR_INVALID_ARG      # in place
    assert L.f3d_unpermute(None, fake, 10, 128, fake, None) == f3d.ERR_INVALID_ARG
    assert L.f3d_unpermute(fake + 1, fake, 10, 128, fake + 4096, None) == f3d.ERR_BAD_ALIGNMENT
    assert L.f3d_unpermute(fake, fake, 0, 128, fake + 4096, None) == f3d.F3D_OK


def test_error_strings():
    assert f3d.error_string(0) == "ok"
    for c in (-1, -2, -3, -4, -5):
        assert f3d.error_string(c) not in ("ok", "unknown error code")
    assert f3d.error_string(-99) == "unknown error code"


def test_backward_workspace_has_room_for_the_sums_of_every_workgroup():
    # the most a call can want beside n x heads floats for D: a strip of bucket_cap x head_dim floats for each of up to 256 tasks (scopes and spare
    # scope slots times heads, in eights), where scopes hold 448 rows or more on average and at most an eighth of the slots, and 8, is spare
    size, seen = ctypes.c_size_t(0), 0
    for heads in (1, 2, 3, 4, 5, 8, 16):
        for scans in (1, 2, 3, 8, 40):
            for n in sorted({int(scans * 448 * 1.13 ** e) for e in range(52)}):
                for cap in (520, 1024, 1500, 2048):
                    for stride in (0, 1, 2, 7, 16):     # 0: plain
                        scan, m = -(-n // scans), 4
                        buckets = -(-scan * m // cap)
                        rest = buckets % (m * stride) if stride else 0
                        scopes = buckets // (m * stride) * stride + min(rest, stride) if stride else -(-buckets // m)
                        slots = (n * m // cap + scans) // m + (stride + 1 if stride else 2) * scans + 1
                        tasks, filled = -(-slots * heads // 8) * 8, scopes * scans * heads
                        if scan // scopes < 448 or tasks <= 128 or tasks > filled + filled // 8 + 8:
                            continue
                        assert f3d.lib().f3d_attn_bwd_workspace_bytes(n, heads, ctypes.byref(size)) == 0
                        assert size.value >= (4 * n * heads + 255) // 256 * 256 + min(tasks, 256) * cap * 32 * 4, (n, heads, scans, cap, stride)
                        seen += 1
    assert seen > 1000
    for n, heads, room in ((50000, 1, 0), (1 << 20, 8, 64 << 20)):   # none below a half round of tasks; a strip per compute unit at most
        assert f3d.lib().f3d_attn_bwd_workspace_bytes(n, heads, ctypes.byref(size)) == 0
        assert size.value == (4 * n * heads + 255) // 256 * 256 + room


def test_product_package_never_touches_the_oracle():
    pkg = os.path.join(ROOT, "paper_2412_16481_amd")
    for dirpath, _, files in os.walk(pkg):
        for fn in files:
            if fn.endswith((".py", ".hip", ".h")):
                text = open(os.path.join(dirpath, fn)).read()
                assert "import oracle" not in text and "from oracle" not in text and "orc_" not in text, fn


def test_binding_refuses_tensors_the_library_could_not_address():
    """The binding hands raw addresses to the C ABI, so it checks device, layout, dtype and shape first (no GPU needed:
    the checks run before any library call)."""
    import torch
    p = f3d.make_params(0.05, 256)
    with pytest.raises(ValueError, match="coords"):
        f3d.psh_bucketize(torch.zeros(10, 3), None, p)                       # host memory
    bk = f3d.Buckets(None, None, None, None, None, 10, 1, 256, 4, 1)
    with pytest.raises(TypeError):
        f3d.bucket_swin_attn(*(torch.zeros(10, 32) for _ in range(3)), bk, 2, 16)   # float32 features
    with pytest.raises(ValueError, match="q must be a contiguous CUDA tensor"):
        f3d.bucket_swin_attn(*(torch.zeros(10, 32, dtype=torch.bfloat16) for _ in range(3)), bk, 2, 16)
    with pytest.raises(ValueError, match="x must be"):
        f3d.ln_linear(torch.zeros(4, 64, dtype=torch.bfloat16), torch.zeros(64, 64, dtype=torch.bfloat16))
    with pytest.raises(ValueError, match="coords"):
        f3d.inbucket_pool(torch.zeros(4, 3), None, torch.zeros(4, 8, dtype=torch.bfloat16), None, 64, 2, 0.1)
    with pytest.raises(ValueError, match="src"):
        f3d.unpermute(torch.zeros(4, 8), torch.zeros(4, dtype=torch.int32))
