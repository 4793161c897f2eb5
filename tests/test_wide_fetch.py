"""Direct loads that share an M0: what the built library may not do in between."""
import re

from .util import device_listing, kernel_bodies


def test_only_the_fetches_write_m0(tmp_path):
    """The 256-row kernels set M0, the LDS address of their direct loads, once for four of them, in an assembly statement ahead of the first.
    That is sound while nothing the compiler makes writes M0: every write in the built code is one of those statements, which end in a
    no-op, and every direct load stands behind one in its kernel."""
    shared = {}
    for kernel, body in kernel_bodies(device_listing(tmp_path)).items():
        written = False
        for at, (line, _) in enumerate(body):
            if re.match(r"s_\w+ m0,", line):
                assert re.match(r"s_(mov_b32 m0, \S+|add_u32 m0, \S+, \S+)$", line) and body[at + 1][0] == "s_nop 0", (kernel, line)
                written = True
            elif re.match(r"global_load_lds_|buffer_load_\w+ .* lds\b", line):
                assert written, (kernel, line)
                if body[at - 1][0] != "s_nop 0":
                    shared[kernel] = shared.get(kernel, 0) + 1
            else:
                assert not re.search(r"\bm0\b", line), (kernel, line)
    # those with 256-row tiles (fourth template argument 2) and no others
    assert len(shared) == 4 and all(re.match(r"void sawattn::attn_fwd_kernel<128, \w+, \w+, 2,", k) for k in shared), shared
