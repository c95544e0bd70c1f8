"""Host-side checks of the C ABI that need no GPU: the library loads, exports every symbol the
header declares, and rejects bad arguments before touching HIP."""
import ctypes
import os
import random
import re
import subprocess

import pytest
import torch

from paper_2507_19906_amd import binding as cd

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def good(**kw):
    base = dict(dtype=cd.BF16, batch=2, n_q_heads=32, n_kv_heads=8, head_dim=128, window=32,
                budget=512, pool_kernel=7)
    base.update(kw)
    return cd.make_params(**base)


def test_header_symbols_are_exported():
    hdr = open(os.path.join(ROOT, "include", "calidrop.h")).read()
    hdr = re.sub(r"/\*.*?\*/", "", hdr, flags=re.S)
    names = set(re.findall(r"\b(calidrop_[a-z_]+)\s*\(", hdr))
    assert {"calidrop_compress", "calidrop_decode", "calidrop_last_error",
            "calidrop_compress_workspace_bytes", "calidrop_decode_workspace_bytes",
            "calidrop_compress_workspace_region", "calidrop_version",
            "calidrop_recalibrate", "calidrop_recalibrate_workspace_bytes"} <= names
    L = cd.lib()
    for n in names:
        assert hasattr(L, n), n
    assert L.calidrop_version() >= 100
    assert ctypes.sizeof(cd.Params) == 56


def test_workspace_sizes():
    p = good()
    n1 = cd.calidrop_compress_workspace_bytes(p, 2 * 8192, 8192)
    n2 = cd.calidrop_compress_workspace_bytes(p, 2 * 32768, 32768)
    assert 0 < n1 < n2 and n1 % 256 == 0
    assert cd.calidrop_decode_workspace_bytes(p, 512) > 0
    off, nbytes = cd.calidrop_compress_workspace_region(p, 2 * 8192, 8192, cd.REGION_SCORE)
    assert nbytes == 2 * 8192 * 8 * 4 and off % 256 == 0 and off + nbytes <= n1
    off, nbytes = cd.calidrop_compress_workspace_region(p, 2 * 8192, 8192, cd.REGION_ROW_LSE)
    assert nbytes == 2 * 8 * 128 * 4


@pytest.mark.parametrize("kw", [
    dict(batch=1), dict(batch=1, dtype=cd.FP32), dict(batch=1, n_q_heads=8, n_kv_heads=8, window=16), dict(batch=2, head_dim=64),
    dict(batch=1, n_q_heads=2, n_kv_heads=1), dict(batch=3, n_q_heads=40), dict(batch=7, window=64, dtype=cd.FP32), dict(batch=64),
    dict(batch=1, n_q_heads=16, n_kv_heads=1, window=100), dict(batch=1, n_q_heads=3, n_kv_heads=3, window=300),
    dict(batch=1, flags=cd.OPT_WIDE_SELECTION), dict(batch=20, pool_kernel=17, n_kv_heads=32)])
def test_a_workspace_for_long_prompts_serves_shorter_ones(kw):
    p = good(**kw)
    nb = p.batch
    recal = [cd.calidrop_recalibrate_workspace_bytes(p, n) for n in range(1, 42000, 37)]
    assert recal == sorted(recal) and min(recal) > 0
    given = [cd.calidrop_compress_given_workspace_bytes(p, n) for n in range(16300, 16500)]
    assert given == sorted(given)
    # every prompt the longest; one long and the others short; lengths in between
    for total in (lambda n: nb * n, lambda n: n + nb - 1, lambda n: n + (nb - 1) * n // 2):
        for lens in (range(1, 42000, 41), range(16200, 16700, 3), range(130900, 131400, 7)):
            for size in ([cd.calidrop_compress_workspace_bytes(p, total(n), n) for n in lens],
                         [cd.calidrop_compress_h2o_workspace_bytes(p, 0, total(n), n) for n in lens]):
                assert size == sorted(size) and size[0] > 0
    rng = random.Random(3)
    for _ in range(3000):
        big = rng.randint(2, 200000)
        small = rng.randint(1, big)
        tot_big = rng.randint(big, nb * big)
        tot_small = rng.randint(small, min(nb * small, tot_big))
        assert cd.calidrop_compress_workspace_bytes(p, tot_small, small) <= cd.calidrop_compress_workspace_bytes(p, tot_big, big)


@pytest.mark.parametrize("kw", [dict(batch=1), dict(batch=1, dtype=cd.FP32, head_dim=64), dict(batch=3, n_q_heads=40), dict(batch=16),
                                dict(batch=64), dict(batch=1, n_q_heads=2, n_kv_heads=1)])
def test_a_workspace_for_long_caches_serves_shorter_ones(kw):
    # 8 KV heads: 4096 rows are 32 splits of 128, 4097 are 17 of 256
    p = good(**kw)
    rows = sorted({*range(1, 9000, 7), *range(4090, 4300), *range(9000, 140000, 501)})
    for size in (cd.calidrop_decode_workspace_bytes, cd.calidrop_recalibrate_packed_workspace_bytes):
        got = [size(p, n) for n in rows]
        assert got == sorted(got) and got[0] > 0


@pytest.mark.parametrize("kw,most", [(dict(batch=1), 2), (dict(batch=1, dtype=cd.FP32), 4), (dict(batch=1, n_q_heads=16), 4), (dict(batch=96), 1)])
def test_h2o_workspace_has_room_for_the_shares_its_heads_can_have(kw, most):
    # streams of up to 2560 blocks of 128 rows are shared, by two workgroups in bf16 from 32 heads on: that many planes for the
    # tokens of such a call, or one for all tokens, and row partials (8 bytes) for its rows
    p = good(**kw)
    heads, n = p.batch * p.n_q_heads, 32768
    votes, _ = cd.calidrop_compress_h2o_workspace_region(p, 0, n * p.batch, n, cd.REGION_VOTE_PLANES)
    score, _ = cd.calidrop_compress_h2o_workspace_region(p, 0, n * p.batch, n, cd.REGION_SCORE)
    plane = max(n * p.batch, most * (2560 * 128 // p.n_q_heads + 1)) * 4 * p.n_q_heads
    parts = most * 8 * (2560 * 128 + heads * 256) if most > 1 else 0
    assert score - votes <= plane + parts + 4096 * p.n_q_heads


@pytest.mark.parametrize("lens,budget", [([1024] * 512, 512), ([600] * 4096, 512), ([8192], 512), ([32768 + 32], 2000)])
def test_short_prompts_carry_no_histograms(lens, budget):
    # the multi-workgroup selection's histograms (50 KiB per KV head, 2 KiB per 8192 positions of one) belong to the calls
    # that run it: prompts beyond 32768 candidates, wide pooling, or on demand
    kw = dict(batch=len(lens), budget=budget)
    args = (sum(lens), max(lens))
    heads = len(lens) * 8
    extra = heads * 4 * ((3 * 4096 + 512) + -(-(max(lens) - 32) // 8192) * 516)
    size = cd.calidrop_compress_workspace_bytes(good(**kw), *args)
    for wide in (dict(flags=cd.OPT_WIDE_SELECTION), dict(pool_kernel=17)):
        assert 0 <= cd.calidrop_compress_workspace_bytes(good(**kw, **wide), *args) - size - extra <= 512
    if max(lens) == 32768 + 32:                      # one candidate more than one workgroup selects from
        assert cd.calidrop_compress_workspace_bytes(good(**kw), args[0] + 1, args[1] + 1) >= size + extra
    h2o = cd.calidrop_compress_h2o_workspace_bytes
    assert 0 <= h2o(good(**kw, flags=cd.OPT_WIDE_SELECTION), 32, *args) - h2o(good(**kw), 32, *args) - extra <= 512


TOOLS = "/opt/rocm/llvm/bin/"
needs_object_tools = pytest.mark.skipif(not os.path.exists(TOOLS + "clang-offload-bundler"), reason="needs the ROCm object tools")


def code_object(lib, tmp_path):
    """The gfx950 code object inside a library built here, as a file."""
    fat, code = str(tmp_path / "fat"), str(tmp_path / "code")
    subprocess.run([TOOLS + "llvm-objcopy", "--dump-section", ".hip_fatbin=" + fat, lib, os.devnull], check=True)
    subprocess.run([TOOLS + "clang-offload-bundler", "--unbundle", "--type=o", "--input=" + fat, "--output=" + code,
                    "--targets=hipv4-amdgcn-amd-amdhsa--gfx950"], check=True)
    return code


def kernel_registers(lib, tmp_path):
    """{mangled kernel name: (vector registers, spilled ones)} from the code object's metadata."""
    notes = subprocess.run([TOOLS + "llvm-readelf", "--notes", code_object(lib, tmp_path)], check=True, capture_output=True,
                           text=True).stdout
    out = {}
    for block in re.split(r"\n\s+- \.agpr_count", notes)[1:]:
        field = lambda k: re.search(r"\." + k + r":\s+(\S+)", block).group(1)
        out[field("name")] = (int(field("vgpr_count")), int(field("vgpr_spill_count")))
    return out


@needs_object_tools
def test_kernels_keep_their_registers(tmp_path):
    # 512 registers a lane and SIMD: what a kernel may use so that the workgroups it counts on fit a compute unit
    regs = kernel_registers(cd.LIB_PATH, tmp_path)
    assert len(regs) > 40 and all(spilled == 0 for _, spilled in regs.values()), {k: v for k, v in regs.items() if v[1]}
    (votes,) = [v for k, v in regs.items() if "h2o_votes_kernelIfLi128ELi2" in k]
    assert votes[0] <= 512 // 3 // 8 * 8
    (select,) = [v for k, v in regs.items() if "select_lds_kernelILi1024ELi8" in k]
    assert select[0] <= 512 // 8                     # two workgroups of 1024 threads


@needs_object_tools
def test_streamed_rows_bypass_the_caches(tmp_path):
    # every 16-byte load of K and V in the streaming passes carries the non-temporal hint; without it are the pieces of the
    # query, in the launches that carry the gather one K and one V piece of a retained row, and in the variant for small
    # passes the two 16-row halves of a wave's first K tile
    asm = subprocess.run([TOOLS + "llvm-objdump", "-d", "--no-show-raw-insn", code_object(cd.LIB_PATH, tmp_path)], check=True,
                         capture_output=True, text=True).stdout
    seen = 0
    for head, body in re.findall(r"^[0-9a-f]+ <(_ZN2cd21attend_partial_kernelI[^>]*)>:\n(.*?)(?=^\S|\Z)", asm, re.M | re.S):
        elem, d, logits, gather, keep = re.search(r"kernelI(f|NS_6bf16_tE)Li(\d+)ELb(\d)ELb\dELb(\d)ELb\dELb(\d)E", head).groups()
        loads = [l for l in body.splitlines() if "global_load_dwordx4" in l]
        pieces = int(d) * (4 if elem == "f" else 2) // 64
        assert sum(" nt" not in l for l in loads) == (0 if logits == "1" else pieces) + 2 * int(gather) + 2 * pieces * int(keep), head
        seen += 1
    assert seen == 32


@pytest.mark.skipif(not os.path.exists("/opt/rocm/bin/hipcc"), reason="needs hipcc")
def test_short_division_rounds_as_the_division_does(tmp_path):
    # the pooled score is sum / k: every significand, for every pooling width of the single-workgroup selection, at 1 and at both
    # ends of the range in which it divides so; without the correction, from a reciprocal one ulp off, some must differ
    src, exe = tmp_path / "divide.hip", tmp_path / "divide"
    src.write_text(f'''
#include "{ROOT}/paper_2507_19906_amd/csrc/cd_select.h"
#include <cstdio>
#include <cstring>
#include <thread>
#include <vector>
static long wrong[cd::kSelMaxPool + 1][2];
static void check(int width) {{
  const float k = static_cast<float>(width), rk = 1.f / k;
  uint32_t bits;
  memcpy(&bits, &rk, 4);
  bits += 1;
  float off;
  memcpy(&off, &bits, 4);
  for (uint32_t base : {{cd::kDivideLow, 127u << 23, cd::kDivideHigh - (1u << 23)}})
    for (uint32_t i = 0; i < (1u << 23); ++i) {{
      const uint32_t u = base + i;
      float s;
      memcpy(&s, &u, 4);
      wrong[width][0] += cd::divide_small(s, k, rk) != s / k;
      wrong[width][1] += base == (127u << 23) && s * off != s / k;
    }}
}}
int main() {{
  std::vector<std::thread> t;
  for (int width = 1; width <= cd::kSelMaxPool; width += 2) t.emplace_back(check, width);
  for (auto& x : t) x.join();
  for (int width = 1; width <= cd::kSelMaxPool; width += 2) printf("%d %ld %ld\\n", width, wrong[width][0], wrong[width][1]);
}}
''')
    subprocess.run(["/opt/rocm/bin/hipcc", "--offload-arch=gfx950", "-O2", "-std=c++17", "-pthread", "-Xarch_host", "-mfma", "-Xarch_host",
                    "-ffp-contract=off", "-w", str(src), "-o", str(exe)], check=True)
    rows = [[int(x) for x in l.split()] for l in subprocess.run([str(exe)], check=True, capture_output=True, text=True).stdout.splitlines()]
    assert [r[0] for r in rows] == list(range(1, 16, 2))
    assert all(r[1] == 0 and r[2] > 0 for r in rows), rows


@pytest.mark.parametrize("lens,heads,w,dtype", [
    ([131072], 8, 64, "bf16"), ([131200], 8, 64, "bf16"), ([140000], 8, 64, "bf16"), ([8192], 8, 32, "bf16"), ([500], 2, 16, "fp32"),
    ([32768] * 32, 8, 32, "bf16"), ([13804] * 13, 2, 32, "fp32"), ([3000] * 20, 8, 64, "fp32"), ([2816, 2816, 2816], 1, 8, "fp32"), ([20000] * 4, 8, 32, "fp32"),
    ([16384, 9000, 13300, 12100, 9900, 16000], 8, 64, "fp32"), ([1200 - 10 * b for b in range(60)], 8, 64, "fp32"),
    ([16384 - 190 * b for b in range(64)], 8, 32, "bf16"), ([4194, 2641, 3000, 3300, 3600, 4000], 8, 64, "fp32")])
def test_scoring_chunks_fill_the_compute_units_with_what_is_launched(lens, heads, w, dtype):
    # the cost of a plan, from the workgroups the lengths really launch: those of the fullest of 256 compute units times
    # the 64-key units of one and what it takes to start; no chunk length that is allowed may be clearly better
    p = cd.make_params(dtype=cd.BF16 if dtype == "bf16" else cd.FP32, batch=len(lens), n_q_heads=4 * heads, n_kv_heads=heads,
                       head_dim=128, window=w, budget=w + 8, pool_kernel=7)
    block = 256 if 4 * w > 128 else 128
    rows = len(lens) * heads * block
    _, nbytes = cd.calidrop_compress_workspace_region(p, sum(lens), max(lens), cd.REGION_ROW_PARTS)
    nch = nbytes // (rows * 8)
    assert nbytes == rows * 8 * nch
    ceil = lambda a, b: -(-a // b)
    even = len(set(lens)) == 1

    def cost(units):
        groups = sum(ceil(n, 64 * units) for n in lens) * heads
        full = ceil(groups, 256)
        if not even:
            load = max(0.25 * full + 0.75 * (groups / 256 + 0.5), 1 if block == 256 else 2)
        else:                                        # 128 rows: a unit holds 4 (fp32: 3), one left over takes the time of two
            load = full if block == 256 else max(full + (full % (4 if dtype == "bf16" else 3) == 1), 2 if dtype == "bf16" else 3)
        return load * (units + 0.5)

    most = 32 if block == 256 else 16 if even else 8
    taken = ceil(ceil(max(lens), nch), 64)
    assert taken <= most
    assert cost(taken) <= (1.0 if even else 1.15) * min(cost(u) for u in range(1, min(most, ceil(max(lens), 64)) + 1))


@pytest.mark.parametrize("kw,status", [
    (dict(head_dim=96), cd.EUNSUPPORTED),
    (dict(n_q_heads=30), cd.ESHAPE),
    (dict(n_q_heads=34, n_kv_heads=2), cd.EUNSUPPORTED),     # G = 17
    (dict(window=0), cd.EINVAL),
    (dict(budget=32), cd.EINVAL),                            # budget must exceed window
    (dict(pool_kernel=4), cd.EINVAL),
    (dict(pool_kernel=0), cd.EINVAL),
    (dict(theta1=0.9, theta2=0.5), cd.EINVAL),
    (dict(theta1=float("nan")), cd.EINVAL),
    (dict(scale=-1.0), cd.EINVAL),
    (dict(batch=0), cd.EINVAL),
    (dict(dtype=7), cd.EUNSUPPORTED),
    (dict(budget=(1 << 24) + 1), cd.EUNSUPPORTED),
])
def test_bad_params_rejected(kw, status):
    p = good(**kw)
    A = 4096     # fake, aligned, never dereferenced: validation fails first
    rc = cd.lib().calidrop_compress(ctypes.byref(p), A, A, A, A, 2 * 8192, 8192, None, A, A, A, A, A, None, A, A, A, A, 1 << 40, None)
    assert rc == status, cd.calidrop_last_error()
    assert cd.calidrop_last_error() != ""
    rc = cd.lib().calidrop_decode(ctypes.byref(p), A, A, A, A, A, 512, A, A, A, A, None, None, A,
                                  1 << 40, None)
    assert rc == status


def test_bad_struct_size_null_align_workspace():
    A = 4096
    L = cd.lib()
    p = good()
    p.struct_size = 40
    assert L.calidrop_compress(ctypes.byref(p), A, A, A, A, 16384, 8192, None, A, A, A, A, A, None, A, A, A, A, 1 << 40, None) == cd.EINVAL
    p = good()
    assert L.calidrop_compress(None, A, A, A, A, 16384, 8192, None, A, A, A, A, A, None, A, A, A, A, 1 << 40, None) == cd.EINVAL
    # null k
    assert L.calidrop_compress(ctypes.byref(p), A, None, A, A, 16384, 8192, None, A, A, A, A, A, None, A, A, A, A, 1 << 40, None) == cd.EINVAL
    assert "k is NULL" in cd.calidrop_last_error()
    # misaligned v
    assert L.calidrop_compress(ctypes.byref(p), A, A, A + 8, A, 16384, 8192, None, A, A, A, A, A, None, A, A, A, A, 1 << 40, None) == cd.EALIGN
    # workspace too small / missing / misaligned
    need = cd.calidrop_compress_workspace_bytes(p, 16384, 8192)
    assert L.calidrop_compress(ctypes.byref(p), A, A, A, A, 16384, 8192, None, A, A, A, A, A, None, A, A, A, A, need - 1, None) == cd.EWORKSPACE
    assert L.calidrop_compress(ctypes.byref(p), A, A, A, A, 16384, 8192, None, A, A, A, A, A, None, A, A, A, None, 0, None) == cd.EWORKSPACE
    assert L.calidrop_compress(ctypes.byref(p), A, A, A, A, 16384, 8192, None, A, A, A, A, A, None, A, A, A, A + 16, need, None) == cd.EALIGN
    # the variant with the window rows' log-sum-exp supplied: same checks, plus its own pointer
    assert L.calidrop_compress_with_lse(ctypes.byref(p), A, A, A, A, 16384, 8192, A + 4, None, A, A, A, A, A, None, A, A, A, A, need, None) == cd.EALIGN
    assert "win_lse" in cd.calidrop_last_error()
    assert L.calidrop_compress_with_lse(ctypes.byref(p), A, None, A, A, 16384, 8192, A, None, A, A, A, A, A, None, A, A, A, A, need, None) == cd.EINVAL
    assert L.calidrop_compress_with_lse(ctypes.byref(p), A, A, A, A, 16384, 8192, A, None, A, A, A, A, A, None, A, A, A, A, need - 1, None) == cd.EWORKSPACE
    # inconsistent sizes
    assert L.calidrop_compress(ctypes.byref(p), A, A, A, A, 100, 8192, None, A, A, A, A, A, None, A, A, A, A, 1 << 40, None) == cd.ESHAPE
    assert L.calidrop_compress(ctypes.byref(p), A, A, A, A, 3 * 8192, 8192, None, A, A, A, A, A, None, A, A, A, A, 1 << 40, None) == cd.ESHAPE      # batch*max < total
    # decode
    needd = cd.calidrop_decode_workspace_bytes(p, 512)
    assert L.calidrop_decode(ctypes.byref(p), A, A, A, A, A, 512, A, A, A, A, None, None, A,
                             needd - 1, None) == cd.EWORKSPACE
    assert L.calidrop_decode(ctypes.byref(p), A, A, A, A, A, 0, A, A, A, A, None, None, A, needd,
                             None) == cd.ESHAPE
    assert L.calidrop_decode(ctypes.byref(p), A, A, A, A, A, 512, A, A, A, None, None, None, A,
                             needd, None) == cd.EINVAL
    # cache_offsets may be NULL (uniform capacity): validation goes on to the next check ...
    assert L.calidrop_decode(ctypes.byref(p), A, A, A, None, A, 512, A, A, A, A, None, None, A,
                             needd - 1, None) == cd.EWORKSPACE
    assert L.calidrop_decode(ctypes.byref(p), A, A, A, A + 4, A, 512, A, A, A, A, None, None, A,
                             needd, None) == cd.EALIGN
    # ... unless the implied token offsets batch * max_cache_len leave the int32 range
    big = good(batch=4096)
    assert L.calidrop_decode(ctypes.byref(big), A, A, A, None, A, 1 << 20, A, A, A, A, None, None, A,
                             1 << 40, None) == cd.EUNSUPPORTED
    assert "uniform" in cd.calidrop_last_error()
    with pytest.raises(cd.CalidropError):
        cd.calidrop_compress_workspace_bytes(good(head_dim=100), 16384, 8192)
    # recalibrate
    needr = cd.calidrop_recalibrate_workspace_bytes(p, 8192)
    assert needr > 0 and needr % 256 == 0
    args = [A, A, A, A, 16384, 8192, A, None, A, A, A, A, A, A]
    assert L.calidrop_recalibrate(ctypes.byref(p), *args, A, needr - 1, None) == cd.EWORKSPACE
    args[8] = None                                          # flags is required here
    assert L.calidrop_recalibrate(ctypes.byref(p), *args, A, needr, None) == cd.EINVAL
    assert "flags is NULL" in cd.calidrop_last_error()
    args[8] = A; args[1] = A + 4
    assert L.calidrop_recalibrate(ctypes.byref(p), *args, A, needr, None) == cd.EALIGN
    assert L.calidrop_recalibrate(ctypes.byref(good(head_dim=96)), A, A, A, A, 16384, 8192, A, None, A, A, A, A, A, A,
                                  A, needr, None) == cd.EUNSUPPORTED
    # calibration size: the list of the calibration set becomes a required argument
    pc = good(calib_size=64)
    args = [A, A, A, A, 16384, 8192, A, None, A, A, A, A, A, A]
    assert L.calidrop_recalibrate(ctypes.byref(pc), *args, A, needr, None) == cd.EINVAL
    assert "cal_indices" in cd.calidrop_last_error()
    assert L.calidrop_compress(ctypes.byref(pc), A, A, A, A, 16384, 8192, None, A, A, A, A, A, None, A, A, A, A,
                               1 << 40, None) == cd.EINVAL
    assert L.calidrop_compress(ctypes.byref(good(calib_size=-1)), A, A, A, A, 16384, 8192, None, A, A, A, A, A, A, A,
                               A, A, A, 1 << 40, None) == cd.EINVAL


def test_older_params_layout_is_accepted():
    # a caller compiled against the 48-byte struct (no calib_size) keeps working
    p = good()
    p.struct_size = 48
    p.calib_size = 12345            # must be ignored: it lies outside the declared size
    assert cd.calidrop_decode_workspace_bytes(p, 512) > 0
    assert cd.calidrop_compress_workspace_bytes(p, 16384, 8192) == cd.calidrop_compress_workspace_bytes(good(), 16384, 8192)
    A = 4096
    # no cal_indices needed: calib_size is 0 for this layout
    need = cd.calidrop_compress_workspace_bytes(p, 16384, 8192)
    assert cd.lib().calidrop_compress(ctypes.byref(p), A, A, A, A, 16384, 8192, None, A, A, A, A, A, None, A, A, A,
                                      A, need - 1, None) == cd.EWORKSPACE


def test_layout_without_flags_is_accepted_and_unknown_flags_are_rejected():
    # a caller compiled against the 52-byte struct (calib_size, no flags) keeps working: flags reads as 0
    p = good(calib_size=7)
    p.struct_size = 52
    p.flags = 0xFFFF                # must be ignored: it lies outside the declared size
    assert cd.calidrop_decode_workspace_bytes(p, 512) > 0
    A = 4096
    assert cd.lib().calidrop_compress(ctypes.byref(p), A, A, A, A, 16384, 8192, None, A, A, A, A, A, None, A, A, A,
                                      A, 1 << 40, None) == cd.EINVAL
    assert "cal_indices" in cd.calidrop_last_error()       # calib_size was read, flags were not
    # per-call options: the two defined bits pass, anything else is an error before any launch
    for ok in (0, cd.OPT_WRITE_SCORES, cd.OPT_WIDE_SELECTION, cd.OPT_WRITE_SCORES | cd.OPT_WIDE_SELECTION):
        assert cd.calidrop_compress_workspace_bytes(good(flags=ok), 16384, 8192) > 0
    bad = good(flags=4)
    assert cd.lib().calidrop_compress(ctypes.byref(bad), A, A, A, A, 16384, 8192, None, A, A, A, A, A, None, A, A, A,
                                      A, 1 << 40, None) == cd.EINVAL
    assert "flags" in cd.calidrop_last_error()


def test_given_strategy_entry_points_validate_on_the_host():
    A = 4096
    L = cd.lib()
    p = good()
    need = cd.calidrop_compress_given_workspace_bytes(p, 8192)
    assert need > 0 and need % 256 == 0
    # streaming list: sink count must fit the budget
    assert L.calidrop_streaming_indices(ctypes.byref(p), -1, A, 16384, 8192, A, None) == cd.EINVAL
    assert L.calidrop_streaming_indices(ctypes.byref(p), 513, A, 16384, 8192, A, None) == cd.EINVAL
    assert "n_sink" in cd.calidrop_last_error()
    assert L.calidrop_streaming_indices(ctypes.byref(p), 32, A, 16384, 8192, None, None) == cd.EINVAL
    assert L.calidrop_streaming_indices(ctypes.byref(p), 32, A, 100, 8192, A, None) == cd.ESHAPE
    # compress_given: q_cal is required, calib_size unsupported, workspace checked
    args = [A, A, A, A, 16384, 8192, A, A, A, A, A, A, A, A]
    assert L.calidrop_compress_given(ctypes.byref(p), *args, A, need - 1, None) == cd.EWORKSPACE
    bad = list(args); bad[0] = None
    assert L.calidrop_compress_given(ctypes.byref(p), *bad, A, need, None) == cd.EINVAL
    assert "q_cal is NULL" in cd.calidrop_last_error()
    bad = list(args); bad[6] = A + 4
    assert L.calidrop_compress_given(ctypes.byref(p), *bad, A, need, None) == cd.EALIGN
    assert L.calidrop_compress_given(ctypes.byref(good(calib_size=8)), *args, A, need, None) == cd.EUNSUPPORTED
    assert L.calidrop_compress_given(ctypes.byref(good(head_dim=96)), *args, A, need, None) == cd.EUNSUPPORTED


def test_offload_entry_points_validate_on_the_host():
    A = 4096
    L = cd.lib()
    p = good()
    assert cd.calidrop_packed_rows(p, 400) == 0 and cd.calidrop_packed_rows(p, 512) == 0
    assert cd.calidrop_packed_rows(p, 8192) == 8192 - 512
    assert cd.calidrop_packed_rows(good(calib_size=100), 8192) == 100
    assert cd.calidrop_packed_rows(good(calib_size=100), 560) == 48
    with pytest.raises(cd.CalidropError):
        cd.calidrop_packed_rows(good(head_dim=100), 8192)
    needp = cd.calidrop_pack_evicted_workspace_bytes(p, 8192)
    assert needp > 0 and needp % 256 == 0
    args = [A, A, A, 16384, 8192, A, None, A, A, A, A, A]
    assert L.calidrop_pack_evicted(ctypes.byref(p), *args, A, needp - 1, None) == cd.EWORKSPACE
    bad = list(args); bad[9] = None
    assert L.calidrop_pack_evicted(ctypes.byref(p), *bad, A, needp, None) == cd.EINVAL
    assert "evict_offsets is NULL" in cd.calidrop_last_error()
    assert L.calidrop_pack_evicted(ctypes.byref(good(calib_size=8)), *args, A, needp, None) == cd.EINVAL
    assert "cal_indices" in cd.calidrop_last_error()
    needr = cd.calidrop_recalibrate_packed_workspace_bytes(p, 7680)
    assert needr > 0
    args = [A, A, A, A, A, 7680, A, A, A, A, A, A]
    assert L.calidrop_recalibrate_packed(ctypes.byref(p), *args, A, needr - 1, None) == cd.EWORKSPACE
    bad = list(args); bad[6] = None
    assert L.calidrop_recalibrate_packed(ctypes.byref(p), *bad, A, needr, None) == cd.EINVAL
    bad = list(args); bad[5] = 0
    assert L.calidrop_recalibrate_packed(ctypes.byref(p), *bad, A, needr, None) == cd.ESHAPE
    bad = list(args); bad[1] = A + 2
    assert L.calidrop_recalibrate_packed(ctypes.byref(p), *bad, A, needr, None) == cd.EALIGN


def test_h2o_entry_point_validates_on_the_host():
    A = 4096
    L = cd.lib()
    p = good()
    need = cd.calidrop_compress_h2o_workspace_bytes(p, 0, 16384, 8192)
    assert need > 0 and need % 256 == 0
    assert cd.calidrop_compress_h2o_workspace_bytes(p, 100, 16384, 8192) > 0
    for bad_local in (-1, 512, 4000):
        with pytest.raises(cd.CalidropError):
            cd.calidrop_compress_h2o_workspace_bytes(p, bad_local, 16384, 8192)
    assert "n_local" in cd.calidrop_last_error()
    args = [A, A, A, A, 16384, 8192, A, A, A, A, A, None, A, A, A]
    assert L.calidrop_compress_h2o(ctypes.byref(p), 0, *args, A, need - 1, None) == cd.EWORKSPACE
    assert L.calidrop_compress_h2o(ctypes.byref(p), 512, *args, A, need, None) == cd.EINVAL
    bad = list(args); bad[0] = None
    assert L.calidrop_compress_h2o(ctypes.byref(p), 0, *bad, A, need, None) == cd.EINVAL
    assert "q_full is NULL" in cd.calidrop_last_error()
    bad = list(args); bad[2] = A + 8
    assert L.calidrop_compress_h2o(ctypes.byref(p), 0, *bad, A, need, None) == cd.EALIGN
    assert L.calidrop_compress_h2o(ctypes.byref(good(calib_size=16)), 0, *args, A, need, None) == cd.EINVAL   # cal_indices missing
    assert L.calidrop_compress_h2o(ctypes.byref(good(batch=4096)), 0, A, A, A, A, 4096 * 8192, 8192, A, A, A, A, A, None,
                                   A, A, A, A, 1 << 44, None) == cd.EUNSUPPORTED              # batch * Hq > 65535
    off, nbytes = cd.calidrop_compress_h2o_workspace_region(p, 0, 16384, 8192, cd.REGION_VOTE_PLANES)
    assert nbytes == 16384 * 8 * 4 * 4 and off % 256 == 0 and off + nbytes <= need      # 16384*8 is a multiple of 64
    off, nbytes = cd.calidrop_compress_h2o_workspace_region(p, 0, 16384, 8192, cd.REGION_ROW_LSE)
    assert nbytes == 2 * 32 * 8192 * 4


def test_probe_library_exports_its_header():
    hdr = open(os.path.join(ROOT, "include", "calidrop_probes.h")).read()
    hdr = re.sub(r"/\*.*?\*/", "", hdr, flags=re.S)
    names = set(re.findall(r"\b(calidrop_probe_[a-z_]+)\s*\(", hdr))
    assert names == {"calidrop_probe_stream_read", "calidrop_probe_stream_read_nt", "calidrop_probe_mfma_loop",
                     "calidrop_probe_mfma_valu", "calidrop_probe_stream_read_pieces", "calidrop_probe_stream_read_store"}
    L = ctypes.CDLL(os.path.join(ROOT, "paper_2507_19906_amd", "libcalidrop_probes.so"))
    for n in names:
        assert hasattr(L, n), n
    L.calidrop_probe_stream_read.argtypes = [ctypes.c_void_p, ctypes.c_uint64, ctypes.c_int32, ctypes.c_void_p, ctypes.c_void_p]
    assert L.calidrop_probe_stream_read(None, 1 << 20, 64, 4096, None) == -1          # validation before any launch
    assert L.calidrop_probe_stream_read(4096, (1 << 20) + 16, 64, 4096, None) == -1
    L.calidrop_probe_mfma_loop.argtypes = [ctypes.c_void_p, ctypes.c_int32, ctypes.c_int32, ctypes.c_void_p]
    assert L.calidrop_probe_mfma_loop(None, 8, 8, None) == -1
    L.calidrop_probe_stream_read_pieces.argtypes = L.calidrop_probe_stream_read.argtypes
    assert L.calidrop_probe_stream_read_pieces(4096, (1 << 20) + 16, 8, 4096, None) == -1
    L.calidrop_probe_stream_read_store.argtypes = [ctypes.c_void_p, ctypes.c_void_p] + [ctypes.c_int32] * 3 + [ctypes.c_void_p] * 2
    assert L.calidrop_probe_stream_read_store(4096, None, 8, 8, 5, 4096, None) == -1      # stores asked for, nowhere to put them
    L.calidrop_probe_mfma_valu.argtypes = [ctypes.c_void_p] + [ctypes.c_int32] * 5 + [ctypes.c_void_p]
    assert L.calidrop_probe_mfma_valu(4096, 8, 8, 1, 4, 0, None) == -1             # 0 or 8 vector instructions per pair
    assert L.calidrop_probe_mfma_valu(4096, 8, 8, 0, 0, 0, None) == -1             # nothing to run


def test_append_validates_on_the_host():
    A = 4096
    L = cd.lib()
    p = good()
    assert L.calidrop_append(ctypes.byref(p), A, A, A, A, A, None, None) == cd.EINVAL
    assert "cache_lens is NULL" in cd.calidrop_last_error()
    assert L.calidrop_append(ctypes.byref(p), A + 4, A, A, A, A, A, None) == cd.EALIGN
    assert L.calidrop_append(ctypes.byref(good(head_dim=80)), A, A, A, A, A, A, None) == cd.EUNSUPPORTED


def test_public_headers_are_plain_c99(tmp_path):
    # the boundary is a C ABI: both headers must compile as C (not only as C++), pedantically
    import shutil
    import subprocess
    gcc = shutil.which("gcc")
    if gcc is None:
        pytest.skip("no C compiler")
    src = tmp_path / "abi.c"
    src.write_text('#include "calidrop.h"\n#include "calidrop_probes.h"\n'
                   "int main(void) { calidrop_params p; p.struct_size = (uint32_t)sizeof(p);\n"
                   "  return (int)(sizeof(calidrop_params) != 56u) + (int)p.struct_size * 0; }\n")
    res = subprocess.run([gcc, "-std=c99", "-Wall", "-Wextra", "-Werror", "-pedantic", "-I", os.path.join(ROOT, "include"),
                          "-fsyntax-only", str(src)], capture_output=True, text=True)
    assert res.returncode == 0, res.stderr


@pytest.mark.parametrize("absent", [(), ("cache_offsets",), ("a_lse", "flags"), ("cache_offsets", "a_lse", "flags", "workspace")])
@pytest.mark.parametrize("as_ints", [False, True])
def test_decode_marshals_tensors_addresses_and_nothing_alike(absent, as_ints, monkeypatch):
    names = ["q_t", "k_c", "v_c", "cache_offsets", "cache_lens", "c_q", "c_out", "c_lse", "out", "a_lse", "flags", "workspace"]
    given = {k: None if k in absent else torch.zeros(8) for k in names}
    want = {k: None if t is None else t.data_ptr() for k, t in given.items()}
    size = 0 if given["workspace"] is None else 32
    seen = []
    fake = type("Lib", (), {"calidrop_decode": staticmethod(lambda *a: seen.append(a) or cd.OK)})
    monkeypatch.setattr(cd, "_lib", fake)
    args = {k: want[k] if as_ints and k != "workspace" else given[k] for k in names}
    cd.calidrop_decode(cd.Params(), max_cache_len=77, stream=5, **args)
    (got,) = seen
    w = [want[k] for k in names]
    assert list(got[1:]) == w[:5] + [77] + w[5:] + [size, 5]


def test_decode_is_told_how_many_rows_live(monkeypatch):
    # params.budget of the decode call: what a compressed cache holds at least, as far as the host knows
    p = good(batch=2, budget=300)
    bufs = cd.CompressBuffers(p, [1000, 200], "cpu", extra_capacity=10)
    short = cd.CompressBuffers(p, [150, 10], "cpu", extra_capacity=10)
    tiny = cd.CompressBuffers(p, [5, 5], "cpu")
    seen = []
    fake = type("Lib", (), {name: staticmethod(lambda par, *a, n=name: seen.append((n, par._obj.budget, par._obj.theta1)) or cd.OK)
                            for name in ("calidrop_decode", "calidrop_append", "calidrop_compress")})
    monkeypatch.setattr(cd, "_lib", fake)
    q = torch.zeros(2, 32, 128, dtype=torch.bfloat16)

    def told(b):
        seen.clear()
        b.decode(q, stream=5)
        return seen[-1][1]

    assert told(bufs) == 300 and told(short) == 150
    for _ in range(3):
        bufs.append(q, q, stream=5)
        short.append(q, q, stream=5)
    assert told(bufs) == 303 and told(short) == 153
    p.theta1 = 0.25                                       # whatever else the caller sets later still arrives
    assert told(bufs) == 303 and seen[-1][2] == 0.25
    for _ in range(9):
        bufs.append(q, q, stream=5)
    assert told(bufs) == 310                              # full
    bufs.compress(q, q, q, q, stream=5)
    assert told(bufs) == 300 and p.budget == 300
    assert told(tiny) == p.window + 1                     # a budget within the window would be refused
