"""CPU check of the rule by which a query's kernel writes an output in place."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SRC = r"""
#include "mp_place.hpp"
#include <cstdio>
int main() {
    const hipMemoryType types[] = {hipMemoryTypeHost, hipMemoryTypeDevice, hipMemoryTypeManaged, hipMemoryTypeUnregistered};
    for (hipMemoryType t : types)
        for (int device : {0, 1})
            for (int own : {0, 1}) {
                hipPointerAttribute_t a = {};
                a.type = t;
                a.device = device;
                std::printf("%d", mp_in_place(a, own) ? 1 : 0);
            }
    return 0;
}
"""


def test_outputs_on_another_device_are_not_written_in_place(tmp_path):
    src, exe = tmp_path / "place.cpp", tmp_path / "place"
    src.write_text(SRC)
    subprocess.run(["g++", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                    "-I" + os.path.join(ROOT, "paper_2404_16370_amd", "csrc"), str(src), "-o", str(exe)], check=True)
    out = subprocess.run([str(exe)], check=True, capture_output=True, text=True).stdout
    # (device, filter's device) = (0, 0), (0, 1), (1, 0), (1, 1): host, device, managed, unknown
    assert out == "0000" + "1001" + "1111" + "0000"
