"""What lanes of a wave hand each other through LDS, seen in the compiler's intermediate code (no GPU): the compiler looks at one lane at a
time, and may hand a lane what it stored itself where another lane has changed it since."""
import os
import re
import subprocess

from paper_2604_02525_amd import build

SNIPPET = """
#include "common.h"
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef u32x4 lds16_t __attribute__((may_alias));
__global__ void k(const u32x4 *x, const int *idx, u32x4 *out)
{
    __shared__ __attribute__((aligned(16))) uint16_t raw[512];
    lds16_t *const own = reinterpret_cast<lds16_t *>(raw + threadIdx.x * 8);
    own[0] = x[threadIdx.x];
    adahop::lds_between_lanes();
    const int at = idx[threadIdx.x];
    if (at >= 0) raw[at] = 0;
    adahop::lds_between_lanes();
    out[threadIdx.x] = own[0];
}
"""


def intermediate(source, *flags):
    cmd = [build.hipcc()] + build.FLAGS + ["-I" + build.CSRC, "--cuda-device-only", "-S", "-emit-llvm", *flags, str(source), "-o", "-"]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    return r.stdout


def test_a_lane_reads_back_what_other_lanes_may_have_changed(tmp_path):
    """The last read stands behind the branch, for all lanes alike: merged from two paths it is a read for one of them only."""
    src = tmp_path / "exchange.hip"
    src.write_text(SNIPPET)
    body = re.search(r"define .*?amdgpu_kernel.*?\n}", intermediate(src), re.S)[0]
    reads = re.findall(r"= load <4 x i32>, ptr addrspace\(3\)", body)
    assert len(reads) == 1 and "phi <4 x i32>" not in body, body


def test_the_quantiser_that_takes_k_channels_out_says_so():
    """Every instance: between a lane's own elements, stored, and the elements taken out of them by whichever lane found their index; and before
    they are read back."""
    code = intermediate(os.path.join(build.CSRC, "quantize.hip"), "-Xclang", "-disable-llvm-passes")
    bodies = [b for b in re.findall(r"\ndefine [^\n]*?quant_kc_gather_rowsILi\d+ELb[01]ELb[01]EEEvRKNS0_7quant_tEjPh\(.*?\n}", code, re.S)]
    assert len(bodies) == 20
    for b in bodies:
        # typed accesses of 16 bytes (copies of a local variable's have no type of their own), and the calls
        seen = "".join("c" if "lds_between_lanes" in m else m[0] for m in re.findall(r"(?:load|store) <4 x i32>[^\n]*!tbaa|call void @\S*lds_between_lanes", b))
        seen = seen[seen.index("c") - 4:]       # l s l s: the two pieces, read from the loaded ones or zero and stored
        assert seen[:6] == "lslscc" and seen[6] == "l" and seen[8] == "l", seen


def test_the_store_of_a_bf16_tile_says_so():
    """Both instances that turn the tile through a wave's patch: between its writes and reads, and before it is written again."""
    code = intermediate(os.path.join(build.CSRC, "gemm_mx.hip"), "-Xclang", "-disable-llvm-passes")
    bodies = re.findall(r"\ndefine [^\n]*@_ZN6adahop12_GLOBAL__N_110store_tileItLNS0_7store_tE[01]E[^\n]*\n.*?\n}", code, re.S)
    assert [len(re.findall(r"call void @\S*lds_between_lanes", b)) for b in bodies] == [2, 2]
