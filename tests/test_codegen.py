"""What the device code has to say in so many words rather than leave to the compiler: small kernels around the library's device
functions are compiled (no GPU needed) and their instructions looked at."""
import collections
import re
import subprocess

import pytest


def _instructions(tmp_path, source, *flags):
    """{kernel: Counter of instructions, with their cache policy bits} of a translation unit beside the library's own"""
    from paper_2010_13887_amd import build as B
    src = tmp_path / "unit.hip"
    src.write_text(source)
    out = tmp_path / "unit.s"
    r = subprocess.run([B._hipcc(), *B.FLAGS, *flags, "-I", B.CSRC, "--cuda-device-only", "-S", str(src), "-o", str(out)],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-3000:]
    found, name = {}, None
    for line in out.read_text().splitlines():
        if m := re.match(r"(\w+):", line):
            name = m.group(1)
        elif name and (m := re.match(r"\s+([a-z]\w+)(.*)", line)):
            policy = " ".join(re.findall(r"\b(sc[01]|nt)\b", m.group(2)))
            found.setdefault(name, collections.Counter())[f"{m.group(1)} {policy}".strip()] += 1
    return found


ROWS = """
#include "search_device.h"
using namespace lsq;
extern "C" __global__ void first_f16(const half_t* e, const float* pe, half_t* x, int d, float s) { embed_row<half_t>(e, pe, x, d, s, threadIdx.x, 64); }
extern "C" __global__ void first_f32(const float* e, const float* pe, float* x, int d, float s) { embed_row<float>(e, pe, x, d, s, threadIdx.x, 64); }
extern "C" __global__ void unscaled_f16(const half_t* e, const float* pe, half_t* x) { embed_whole_row<half_t, 768>(e, pe, x, 1.0f, threadIdx.x); }
extern "C" __global__ void next_f16(NextInput nx, const int* tok, int k, int pos) { next_input_rows<half_t>(nx, tok, 0, k, pos, threadIdx.x); }
extern "C" __global__ void next_f32(NextInput nx, const int* tok, int k, int pos) { next_input_rows<float>(nx, tok, 0, k, pos, threadIdx.x); }
"""


@pytest.mark.parametrize("contract", ["off", "fast"])
def test_input_rows_are_one_arithmetic_whatever_the_compiler_likes(tmp_path, contract):
    """x * scale + p of a decoder input row: one multiply-add, rounded once to the type that is stored, in the kernels that make the
    first step's rows and in those that make every later step's, with and without contraction."""
    found = _instructions(tmp_path, ROWS, f"-ffp-contract={contract}")
    for kernel in ("first_f16", "first_f32", "unscaled_f16", "next_f16", "next_f32"):
        ops = found[kernel]
        loose = [i for i in ops if re.match(r"v_(pk_)?add_f(16|32)|v_cvt_(pk_)?f16_f32|v_cvt_pkrtz", i)]
        assert not loose, (kernel, loose)
        fused = sum(n for i, n in ops.items() if re.match(r"v_fma_mix(lo|hi)_f16" if kernel.endswith("f16") else r"v_(fma|fmac)_f32", i))
        assert fused >= 8, (kernel, ops)


def test_values_published_on_a_die_leave_the_compute_unit(tmp_path):
    """The kernels with a group of rows per die publish with stores of workgroup scope at least: a store without a scope is for the
    wavefront itself, and nothing says when the compute units that poll for it see it."""
    found = _instructions(tmp_path, '#include "kernels_stack_die.hip"\n')
    kernels = [k for k in found if "decoder_die_kernel" in k and any(i.startswith("buffer_load") for i in found[k])]
    assert len(kernels) == 6, list(found)   # groups of 4, 8 and 16 rows, post-LN and pre-LN
    for k in kernels:
        stores = [i for i in found[k] if i.startswith("buffer_store")]
        assert stores and all(" sc" in i for i in stores), (k, stores)
        polls = [i for i in found[k] if i.startswith("buffer_load")]
        assert all("sc1" in i for i in polls), (k, polls)


ATTEND = """
#include "stack_attend.h"
using namespace lsq;
extern "C" __global__ void attend(const half8_t* kv, half_t* out, int n) {
  const int lane = threadIdx.x;
  half8_t kn[kTrip], vn[kTrip];
  for (int u = 0; u < kTrip; ++u) { kn[u] = kv[u * 64 + lane]; vn[u] = kv[(kTrip + u) * 64 + lane]; }
  Attention t;
  auto live = [&](int u) { return u * 8 + (lane >> 3) < n; };
  t.first<true>(kv[1000 + lane], kn, vn, kv[2000 + lane], n == 0, live, [] {});
  t.more(kv[1000 + lane], vn, kn, live, [] {});
  t.add(kv[3000 + lane], lane < 8);
  t.sum<false>();
  *reinterpret_cast<half2_t*>(out + own_column<false>(lane)) = context_of(t.acc[0], t.acc[1], t.z);
}
"""


def test_attention_of_the_stack_kernels_is_one_arithmetic_whatever_the_compiler_likes(tmp_path):
    """Its last bit decides draws: the same multiply-adds with and without contraction, a context divided by the sum of its weights
    with a division, and rounded to float16 after the product."""
    counts = {}
    for contract in ("off", "fast"):
        ops = _instructions(tmp_path, ATTEND, f"-ffp-contract={contract}")["attend"]
        kinds = {"fma": r"v_(fma|fmac|fma_mix)_f32", "mul": r"v_mul_f32", "add": r"v_(add|sub|subrev)_f32", "exp": r"v_exp_f32", "div": r"v_div_fixup_f32"}
        counts[contract] = {k: sum(n for i, n in ops.items() if re.match(p, i)) for k, p in kinds.items()}
        assert not [i for i in ops if i.startswith("v_fma_mix") and "f16" in i], ops
    assert counts["off"] == counts["fast"], counts
    assert counts["fast"]["div"] == 1 and counts["fast"]["exp"] == 4 + 5 + 2, counts


@pytest.mark.parametrize("source,kernels", [("kernels_stack.hip", 30), ("kernels_stack_die.hip", 6)])
def test_float16_stack_kernels_spill_no_vector_register(tmp_path, source, kernels):
    """A layer's matrices wait in registers; what does not fit beside them goes to memory and back in every layer."""
    from paper_2010_13887_amd import build as B
    out = tmp_path / "unit.s"
    r = subprocess.run([B._hipcc(), *B.FLAGS, "-I", B.CSRC, "--cuda-device-only", "-S", f"{B.CSRC}/{source}", "-o", str(out)],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-3000:]
    spilled = {}
    for entry in out.read_text().split("\n  - .")[1:]:
        name = re.search(r"\.name:\s+(\S*decoder_(?:stack|die)\S*)", entry)
        count = re.search(r"\.vgpr_spill_count:\s+(\d+)", entry)
        if name and count:
            spilled[name.group(1)] = int(count.group(1))
    assert len(spilled) == kernels, sorted(spilled)
    assert not any(spilled.values()), spilled


MERGE = """
#include "lsq_internal.h"
using namespace lsq;
extern "C" __global__ void merge(const float* s, float* o) {
  __shared__ float m[4][64], z[4][64];
  const int lane = threadIdx.x;
  for (int w = 0; w < 4; ++w) { m[w][lane] = s[w * 128 + lane]; z[w][lane] = s[w * 128 + 64 + lane]; }
  __syncthreads();
  float mx = m[0][lane ^ 1], sum = z[0][lane ^ 1];
  for (int w = 1; w < 4; ++w) merge_stat_exact(mx, sum, m[w][lane ^ 1], z[w][lane ^ 1]);
  o[lane] = mx;
  o[64 + lane] = sum;
}
"""


def test_statistics_are_merged_in_one_arithmetic_without_a_branch(tmp_path):
    """What two kernels share bit for bit: a multiply-add and a product a merge, with and without contraction, and nothing that waits behind a
    branch for its operands."""
    for contract in ("off", "fast"):
        ops = _instructions(tmp_path, MERGE, f"-ffp-contract={contract}")["merge"]
        assert sum(n for i, n in ops.items() if re.match(r"v_(fma|fmac)_f32", i)) == 3, (contract, ops)
        assert not [i for i in ops if i.startswith("s_cbranch") or "saveexec" in i], (contract, ops)
