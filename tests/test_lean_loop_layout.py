"""Layout of the resident states' rotation loops, in the generator's output and
in the built gfx950 code: a computed jump adds the record's offset, variant
index times a fixed stride, to the table's address, so every variant has to
start at exactly that multiple."""
import importlib.util
import os

import pytest

from test_abi_host import ROOT, _branch_target, _code_object

CSRC = os.path.join(ROOT, "paper_2504_17881_amd", "csrc")


def _gen():
    spec = importlib.util.spec_from_file_location("gen_rot_jump", os.path.join(CSRC, "gen_rot_jump.py"))
    gen = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(gen)
    return gen


def test_loops_are_generated_and_wait_for_their_loads():
    gen = _gen()
    for f64, tile in ((False, False), (True, False), (False, True), (True, True)):
        name = f"rot_lean{'_tile' if tile else ''}_{'f64' if f64 else 'f32'}m4.inc"
        with open(os.path.join(CSRC, name)) as f:
            text = f.read()
        lines = gen.lean_block(f64, tile)
        assert [ln.split('"')[1][:-2] for ln in text.splitlines() if ln.startswith('    "')] == lines
        # the only ways out pass a wait for the record loaded ahead
        assert lines[lines.index("8:") + 1] == "s_waitcnt lgkmcnt(0)"
        assert all(b == "s_waitcnt lgkmcnt(0)" for a, b in zip(lines, lines[1:])
                   if a == "s_cbranch_scc1 8f")
    for block in (gen.loop_block(), gen.loop_block64()):
        assert block[block.index("9:") + 1] == "s_waitcnt lgkmcnt(0)"


@pytest.mark.parametrize("obj_name", ["kernels.hip.o", "batch.hip.o"])
def test_layout_in_built_code(tmp_path, obj_name):
    gen = _gen()
    ins = _code_object(tmp_path, obj_name)
    addr = [a for a, _, _ in ins]
    at = {a: i for i, a in enumerate(addr)}
    jumps = [i for i, (_, op, txt) in enumerate(ins) if op == "s_setpc_b64" and "s[94:95]" in txt]
    heads = [i for i in jumps if any(op == "s_getpc_b64" for _, op, _ in ins[i - 20:i])]
    assert len(jumps) == 65 * len(heads)
    seen = set()
    for i in heads:
        g = max(j for j in range(i - 20, i) if ins[j][1] == "s_getpc_b64")
        assert "s[92:93]" in ins[g][2]
        off = int(ins[g + 1][2].rsplit(",", 1)[1].strip(), 0)
        start = addr[i + 1]
        assert addr[g + 1] + off == start         # the table follows the head's jump
        f64 = ins[i + 2][1] == "s_load_dwordx2"
        tile = any(op == "s_bcnt1_i32_b64" for _, op, _ in ins[g:i])
        stride = (gen.LEAN64_VARIANT_BYTES if f64 else gen.LEAN_VARIANT_BYTES) + 8 * tile
        lead = 2 if f64 else 1
        seen.add(stride)
        end = None
        for var in range(64):
            j = at[start + stride * var]
            assert ins[j][1] == "s_load_dwordx8" and "s[80:87], s[76:77]" in ins[j][2]
            fma = [op for _, op, _ in ins[j + lead:j + lead + 32]]
            assert fma == ["v_fma_f64" if f64 else "v_fma_f32"] * 32
            k = j + lead + 32
            assert ins[k][1] == "s_sub_u32" and ins[k + 1][1] == "s_cbranch_scc1"
            end = end or _branch_target(ins, k + 1)
            assert _branch_target(ins, k + 1) == end
            assert ins[k + 2][1] == "s_waitcnt" and "s92, s85" in ins[k + 3][2]
            assert ins[at[start + stride * (var + 1)] - 1][1] == "s_setpc_b64"
        j = at[start + stride * 64]               # the diagonal entry puts the record back
        size = 40 if f64 else 32
        assert ins[j][1] == "s_sub_u32" and ins[j][2].endswith(f"s76, s76, {size}")
        assert [op for _, op, _ in ins[j + 1:j + 4]] == ["s_subb_u32", "s_add_u32", "s_branch"]
        assert ins[at[end]][1] == "s_waitcnt"
        assert _branch_target(ins, j + 3) == addr[at[end] + 2]
    assert seen == {324, 340, 332, 348}
    # the records' offsets use the same strides
    with open(os.path.join(CSRC, "internal.h")) as f:
        text = f.read()
    assert "sizeof(T) == 4 ? 324u : 340u" in text and "kLeanTileMore = 8u" in text
    assert (gen.LEAN_VARIANT_BYTES, gen.LEAN64_VARIANT_BYTES) == (324, 340)
