"""MFMAs written as assembly: the wait states that the compiler does not add, read from the built library."""
import re

from .util import device_listing, kernel_bodies

# 16x16 MFMAs of 4 passes: their result is there 4 passes and 3 wait states later; what a vector instruction writes is read by an MFMA
# no sooner than 2 wait states later.  Every instruction in between counts as one, s_nop n as n + 1.
RESULT, OPERAND = 7, 2


def registers(text):
    out = set()
    for file, first, last, one_file, one in re.findall(r"\b([va])\[(\d+):(\d+)\]|\b([va])(\d+)\b", text):
        out |= {(file, k) for k in range(int(first), int(last) + 1)} if file else {(one_file, int(one))}
    return out


def is_mfma(op):
    return op.startswith(("v_mfma", "v_smfmac"))


def too_early(body):
    """Pairs of instructions (text, text, wait states between them) of a kernel that stand too close; `body` as kernel_bodies gives it."""
    ops = [text.split(None, 1) + [""] for text, _ in body]
    args = [[registers(a) for a in re.split(r",\s*", op[1])] for op in ops]
    found = []

    def following(i, states, look):
        """Calls look(j, wait states between) for what can run behind instruction i until it says stop."""
        todo, seen = [(i + 1, 0)], set()
        while todo:
            j, w = todo.pop()
            if j >= len(body) or w >= states or (j, w) in seen:
                continue
            seen.add((j, w))
            op, target = ops[j][0], body[j][1]
            if op == "s_endpgm" or look(j, w):
                continue
            if target is not None:
                todo.append((target, w + 1))
            if op != "s_branch":
                todo.append((j + 1, w + (int(ops[j][1], 0) + 1 if op == "s_nop" else 1)))

    for i, (op, *_) in enumerate(ops):
        written = args[i][0]
        if is_mfma(op):
            def look(j, w):
                other = ops[j][0]
                if is_mfma(other):
                    read = args[j][1] | args[j][2]
                    # (an accumulator as a whole may follow on itself)
                    if written & read or (written & args[j][3] and args[j][0] != written):
                        found.append((body[i][0], body[j][0], w))
                    return args[j][0] >= written
                if other.startswith(("v_", "ds_", "global_", "buffer_", "scratch_")) and written & set().union(*args[j]):
                    found.append((body[i][0], body[j][0], w))
                    return True
                return False
            following(i, RESULT, look)
        elif op.startswith("v_"):
            def look(j, w):
                if is_mfma(ops[j][0]) and written & set().union(*args[j][1:]):
                    found.append((body[i][0], body[j][0], w))
                    return True
                return False
            following(i, OPERAND, look)
    return found


def test_the_walk_finds_what_stands_too_close():
    def body(*lines):
        return [(text, None) for text in lines]
    mfma = "v_mfma_f32_16x16x32_f16 v[0:3], v[8:11], a[0:3], 0"
    assert too_early(body("v_cvt_pk_f16_f32 v8, v20, v21", mfma))
    assert too_early(body("v_cvt_pk_f16_f32 v8, v20, v21", "s_barrier", mfma))
    assert not too_early(body("v_cvt_pk_f16_f32 v8, v20, v21", "s_nop 1", mfma))
    assert too_early(body(mfma, "s_nop 5", "v_max3_f32 v30, v30, v1, v2"))
    assert not too_early(body(mfma, "s_nop 6", "v_max3_f32 v30, v30, v1, v2"))
    assert too_early(body(mfma, "v_mfma_f32_16x16x32_f16 a[8:11], v[2:5], v[12:15], a[8:11]"))
    assert not too_early(body(mfma, "v_mfma_f32_16x16x32_f16 v[0:3], v[12:15], a[4:7], v[0:3]"))
    assert too_early([("s_nop 0", None), ("v_max_f32_e32 v9, v0, v0", None), (mfma, None), ("s_cbranch_scc1 65533", 1), ("s_endpgm", None)])


def test_256_row_kernels_keep_their_distances(tmp_path):
    bodies = kernel_bodies(device_listing(tmp_path))
    wide = {k: b for k, b in bodies.items() if re.match(r"void sawattn::attn_fwd_kernel<128, \w+, \w+, 2,", k)}
    assert len(wide) == 4, list(bodies)
    for kernel, body in wide.items():
        assert sum(is_mfma(text) for text, _ in body) > 256, kernel       # 64 + 64 of a tile in the loop and the same around it
        assert not too_early(body), (kernel, too_early(body)[:4])
