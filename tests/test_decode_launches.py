"""Which kernels a decode call launches, and for which it sets the attribute of their LDS: the library linked into a program that brings
its own launch functions and writes down what they are asked for.  No GPU needed, nothing runs on one."""
import os
import subprocess

import pytest

from paper_2605_23258_amd import build

pytestmark = pytest.mark.skipif(not os.path.exists(build.HIPCC), reason="needs the ROCm toolchain")

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PROGRAM = r"""
#include <cstdio>
#include <cstdlib>
#include <map>
#include <string>
#include <vector>
#include "vector.h"
struct dim3 { unsigned x, y, z; };
static std::map<const void*, std::string>& names() { static std::map<const void*, std::string> n; return n; }
static dim3 g_grid, g_block;
static size_t g_lds;
static void* g_stream;
extern "C" {
void** __hipRegisterFatBinary(const void*) { static void* handle; return &handle; }
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterVar(void**, void*, char*, const char*, int, size_t, int, int) {}
void __hipRegisterFunction(void**, const void* f, char*, const char* name, unsigned, void*, void*, void*, void*, int*) { names()[f] = name; }
int __hipPushCallConfiguration(dim3 grid, dim3 block, size_t lds, void* stream) { g_grid = grid; g_block = block; g_lds = lds; g_stream = stream; return 0; }
int __hipPopCallConfiguration(dim3* grid, dim3* block, size_t* lds, void** stream) { *grid = g_grid; *block = g_block; *lds = g_lds; *stream = g_stream; return 0; }
int hipLaunchKernel(const void* f, dim3 grid, dim3 block, void**, size_t lds, void*) {
  printf("launch %s %u %u %u %zu\n", names()[f].c_str(), grid.x, grid.y, grid.z, lds);
  return 0;
}
int hipFuncSetAttribute(const void* f, int, int value) { printf("set %s %d\n", names()[f].c_str(), value); return 0; }
int hipOccupancyMaxActiveBlocksPerMultiprocessor(int* n, const void*, int, size_t lds) { *n = lds > 60000 ? 2 : 3; return 0; }
int hipGetLastError() { return 0; }
}
// sequences, KV heads, query heads per KV head, dims, capacity, approximated rows, capacities of the sequences' own, rotated keys
int main(int, char** v) {
  const int B = atoi(v[1]), H = atoi(v[2]), G = atoi(v[3]), d = atoi(v[4]), cap = atoi(v[5]), apx = atoi(v[6]);
  static char memory[4096] __attribute__((aligned(256)));
  vector_cache c = {};
  c.batch = B; c.n_q_heads = H * G; c.n_kv_heads = H; c.head_dim = d; c.dtype = VECTOR_BF16; c.cap_retain = cap; c.n_approx = apx;
  c.len_retain = (const int32_t*)memory;
  c.k_ret = c.v_ret = c.k_apx = c.W = memory;
  if (atoi(v[7])) { c.cap_retain_seq = c.n_approx_seq = (const int32_t*)memory; c.ret_row_start = c.apx_row_start = (const int64_t*)memory; }
  std::vector<float> freq(64, 1.f);
  vector_rope rope = {};
  for (int i = 0; i < 2; ++i) {
    printf("call\n");
    if (atoi(v[8])) {
      rope.inv_freq = reinterpret_cast<decltype(rope.inv_freq)>(memory);
      if (vector_decode_attn_rope(&c, &rope, memory, 1.f, memory, 0, memory, (size_t)1 << 40, nullptr)) return 1;
    } else if (vector_decode_attn(&c, memory, 1.f, memory, 0, memory, (size_t)1 << 40, nullptr)) {
      return 2;
    }
  }
  return 0;
}
"""


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    if not os.path.exists(build.LIB_PATH):
        build.build_library()
    out = tmp_path_factory.mktemp("launches")
    (out / "launches.cpp").write_text(PROGRAM)
    exe = str(out / "launches")
    subprocess.run([os.path.join(os.path.dirname(build.HIPCC), "amdclang++"), "-std=c++17", "-O1", "-w", "-rdynamic", "-I", os.path.join(ROOT, "include"), str(out / "launches.cpp"),
                    build.LIB_PATH, "-Wl,-rpath," + build.PKG_DIR, "-Wl,-rpath,/opt/rocm/lib", "-L/opt/rocm/lib", "-lamdhip64", "-o", exe], check=True)
    return exe


def second_call(program, *shape):
    r = subprocess.run([program, *map(str, map(int, shape))], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout + r.stderr
    lines = [line.split() for line in r.stdout.split("call\n")[2].splitlines()]
    return [line[1] for line in lines if line[0] == "set"], [line[1:] for line in lines if line[0] == "launch"]


# sequences, KV heads, query heads, dims, capacity, approximated rows, own capacities, rotated keys
SHAPES = [(1, 8, 4, 128, 1075, 819, 0, 0), (16, 8, 4, 128, 3532, 3276, 0, 0), (16, 8, 4, 128, 3532, 3276, 0, 1), (24, 8, 4, 128, 1856, 1600, 1, 0), (24, 8, 4, 128, 1856, 1600, 1, 1),
          (1, 8, 4, 64, 1075, 819, 0, 0), (40, 8, 4, 64, 1856, 1600, 1, 0), (40, 8, 4, 64, 1856, 1600, 1, 1), (2, 2, 16, 128, 1075, 819, 1, 0)]


@pytest.mark.parametrize("shape", SHAPES)
def test_attributes_of_launched_kernels_only(program, shape):
    """An attribute set for a kernel that the call does not launch is host time of every step."""
    attributes, launches = second_call(program, *shape)
    assert len(launches) == 2 and len(set(attributes)) == len(attributes)
    assert set(attributes) <= {name for name, *_ in launches}
    assert all(name in attributes for name, *_, lds in launches if int(lds) > 48 * 1024)


ROTATED, PLANNED, APPLYING = 0, 3, 4          # of the split kernel's five switches


# a capacity of 2^20 rows: as the tests of the plan on small shapes state it
@pytest.mark.parametrize("shape,switches", [
    (SHAPES[0], {APPLYING}), (SHAPES[1], set()), (SHAPES[2], {ROTATED}), (SHAPES[3], {PLANNED}), (SHAPES[4], {ROTATED, PLANNED}), (SHAPES[5], {APPLYING}), (SHAPES[6], {PLANNED}),
    (SHAPES[7], {ROTATED}), (SHAPES[8], set()), ((2, 1, 4, 128, 1 << 20, 0, 1, 0), {PLANNED}), ((2, 2, 4, 128, 1 << 20, 31, 1, 1), {ROTATED, PLANNED}),
    ((4, 3, 16, 64, 1 << 20, 2000, 1, 0), {PLANNED}), ((3, 2, 4, 128, 0, 1 << 20, 1, 0), {PLANNED}), ((65, 1, 4, 128, 1 << 20, 200, 1, 0), set())])
def test_split_kernel(program, shape, switches):
    _, launches = second_call(program, *shape)
    name = launches[0][0].split("decode_split_mfma_kernel")[1]
    assert {i for i, on in enumerate(name.split("ELb")[1:6]) if on[0] == "1"} == switches
