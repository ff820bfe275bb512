"""Which kernel a convolution layer takes, asked without a GPU: the library's own launch_conv in a small program whose launch functions do nothing.
256 compute units, as on MI355X."""
import os
import subprocess

from paper_2502_01277_amd import binding
from paper_2502_01277_amd.build import HERE

ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")
DTYPES = {"f32": 0, "f16": 1, "bf16": 2, "f8": 3}
# place: a layer of a model; split, hint: item counts stated and expected where the count is taken on the device; second: channels of the first of two
# layers in one launch; upsampled: an upsampling of the output follows; bare: of a model, but without what one keeps for conv3x3_held_kernel
FIELDS = ("n", "h", "w", "cin", "cout", "k", "stride", "res", "place", "split", "hint", "second", "upsampled", "bare")

SOURCE = r'''
#include "csrc/conv3x3_held_choice.h"
#include <cstdio>
extern "C" hipError_t hipLaunchKernel(const void*, dim3, dim3, void**, size_t, hipStream_t) { return hipSuccess; }
extern "C" hipError_t hipExtLaunchKernel(const void*, dim3, dim3, void**, size_t, hipStream_t, hipEvent_t, hipEvent_t, int) { return hipSuccess; }
extern "C" hipError_t hipFuncSetAttribute(const void*, hipFuncAttribute, int) { return hipSuccess; }
extern "C" hipError_t hipGetLastError() { return hipSuccess; }
int main() {
  int dt, n, h, w, ci, co, k, st, res, place, split, hint, second, up, bare;
  while (scanf("%d %d %d %d %d %d %d %d %d %d %d %d %d %d %d", &dt, &n, &h, &w, &ci, &co, &k, &st, &res, &place, &split, &hint, &second, &up, &bare) == 15) {
    octo::ConvArgs a{};
    a.x = (void*)0x10000; a.w = (void*)0x20000; a.bias = (float*)0x30000; a.y = (void*)0x40000;      // never followed
    if (res) { a.res = (void*)0x50000; a.res_mode = res; a.res_ld = co; }
    a.n = n; a.H = h; a.W = w; a.Cin = a.x_ld = ci; a.kh = a.kw = k; a.stride_h = a.stride_w = st; a.pad_h = a.pad_w = k / 2;
    a.Ho = (h + 2 * (k / 2) - k) / st + 1; a.Wo = (w + 2 * (k / 2) - k) / st + 1; a.Cout = a.y_ld = co; a.K = k * k * ci;
    octo::conv_packed_weight_elems(co, k, k, ci, dt, &a.Kp, &a.w_rows);
    a.in_place = place; a.n_split = split; a.n_hint = hint; a.up_next = up; a.act = OCTO_ACT_SILU;
    if (split || hint) a.n_dyn = (int*)0x60000;
    if (second) { a.split = a.y_ld = second; a.y2 = (void*)0x70000; a.y2_ld = co - second; }
    octo::HeldPlan plan;
    if (place && !bare && (dt == OCTO_F16 || dt == OCTO_BF16) && octo::held_layer(k, k, st, k / 2, h, ci, co)) {
      plan = octo::held_plan(st, w, a.Ho, a.Wo, ci, co);
      plan.w = (void*)0x90000;
      a.held = &plan;
    }
    if (dt == OCTO_F8) { a.scale = (float*)0x80000; a.res_scale = a.y_inv_scale = 1; }
    int kid = -1;
    const hipError_t e = octo::launch_conv(dt, a, 256, nullptr, &kid);
    printf("%d\n", e == hipSuccess ? kid : -(int)e);
  }
}
'''


def compile_host(args):
    subprocess.run(["g++", "-O1", "-std=c++17", "-w", "-D__HIP_PLATFORM_AMD__", "-I", ROCM + "/include", "-I", HERE] + args, check=True)


def program(folder) -> str:
    """Builds the program; one per test module will do."""
    src, exe = os.path.join(str(folder), "dispatch.cpp"), os.path.join(str(folder), "dispatch")
    with open(src, "w") as f:
        f.write(SOURCE)
    # -rdynamic: the library's calls of the launch functions find those of the program
    compile_host(["-o", exe, src, binding.LIB_PATH, "-rdynamic", "-L", ROCM + "/lib", "-lamdhip64", "-Wl,-rpath," + ROCM + "/lib", "-Wl,-rpath," + HERE])
    return exe


def kernel_ids(exe, layers) -> list:
    """layers: dicts with "dtype" and any of FIELDS (n, h, w, cin and cout are needed).  Per layer the kernel's id, or a negative error."""
    rows = [" ".join([str(DTYPES[l["dtype"]])] + [str(int(l.get(f, 1 if f in ("k", "stride") else 0))) for f in FIELDS]) for l in layers]
    r = subprocess.run([exe], input="\n".join(rows) + "\n", capture_output=True, text=True, check=True)
    ids = [int(v) for v in r.stdout.split()]
    assert len(ids) == len(layers)
    return ids
