"""Direct loads that share an M0: what the built library may not do in between."""
import re
import shutil
import subprocess


def test_only_the_fetches_write_m0(tmp_path):
    """The 256-row kernels set M0, the LDS address of their direct loads, once for four of them, in an assembly statement ahead of the first.
    That is sound while nothing the compiler makes writes M0: every write in the built code is one of those statements, which end in a
    no-op, and every direct load stands behind one in its kernel."""
    from paper_2601_16032_amd import build as hip_build
    objdump = "/opt/rocm/llvm/bin/llvm-objdump"
    shutil.copy(hip_build.LIB_PATH, tmp_path / "lib.so")
    subprocess.run([objdump, "--offloading", "lib.so"], cwd=tmp_path, check=True, capture_output=True)
    device, = tmp_path.glob("lib.so.*gfx950")
    listing = subprocess.run([objdump, "-d", "--mcpu=gfx950", str(device)], check=True, capture_output=True, text=True).stdout.splitlines()
    kernel, shared, written = None, {}, set()
    for at, line in enumerate(listing):
        head = re.match(r"[0-9a-f]+ <(\w+)>:", line)
        if head:
            kernel = head.group(1)
        elif re.match(r"\s*s_\w+ m0,", line):
            assert re.match(r"\s*s_(mov_b32 m0, \S+|add_u32 m0, \S+, \S+)\s", line) and re.match(r"\s*s_nop 0\s", listing[at + 1]), (kernel, line)
            written.add(kernel)
        elif re.search(r"\bm0\b", line.split("//")[0]):
            raise AssertionError((kernel, line))
        elif re.match(r"\s*(global_load_lds_|buffer_load_\w+ .* lds\b)", line):
            assert kernel in written, (kernel, line)
            if not re.match(r"\s*s_nop 0\s", listing[at - 1]):
                shared[kernel] = shared.get(kernel, 0) + 1
    assert len(shared) == 4 and all("attn_fwd_kernel" in k and "ELi2ELb0E" in k for k in shared), shared
