"""The threaded rotation loops wait for the record that they load ahead before
they leave: its registers are the compiler's again from there on."""
import importlib.util
import os

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2504_17881_amd", "csrc")


def _gen():
    spec = importlib.util.spec_from_file_location("gen_rot_jump", os.path.join(CSRC, "gen_rot_jump.py"))
    gen = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(gen)
    return gen


def test_loops_wait_for_their_loads():
    gen = _gen()
    for block in (gen.loop_block(), gen.loop_block64()):
        assert block[block.index("9:") + 1] == "s_waitcnt lgkmcnt(0)"
