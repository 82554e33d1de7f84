"""Which attention calls are divided, and the scratch that they ask for: the library's host arithmetic, no GPU."""
import os
import subprocess

import pytest

from paper_2602_02958_amd import binding as B
from paper_2602_02958_amd import build as qbuild

STATE = 66 * 512 * 4                             # bytes of a query block's state
SHAPES = [(1, 1), (1, 64), (1, 300), (2, 64), (8, 64), (3, 700), (9, 64), (16, 200), (5, 600), (12, 600), (64, 64), (65, 64), (40, 700),
          (12, 1560), (128, 256), (129, 64), (256, 64)]


def _scratch(H, Nq, tiles, lengths=False):
    need, p = B.C.c_size_t(), B.make_params(H, 16, 64, 2)
    ask = B.lib().qvg_attn_scratch_bytes_causal if lengths else B.lib().qvg_attn_scratch_bytes
    assert ask(B.C.byref(p), Nq, tiles * 64 - 3, 1 << 20, B.C.byref(need)) == 0
    return need.value


def _parts_of_four_tiles(blocks, tiles):
    """The parts of a call that has always been divided: four tiles to a part at least, until 256 workgroups are there; of
    more than 64 blocks not below ten tiles."""
    return 1 if blocks > 64 and tiles < 10 else min(256 // blocks, tiles // 4)


@pytest.mark.parametrize("lengths", [False, True])
@pytest.mark.parametrize("H,Nq", SHAPES)
def test_calls_that_were_divided_are(H, Nq, lengths):
    blocks = H * -(-Nq // 256)
    for tiles in range(1, 192):
        if blocks <= 256 and _parts_of_four_tiles(blocks, tiles) > 1:
            assert _scratch(H, Nq, tiles, lengths) >= 2 * blocks * STATE, tiles


@pytest.mark.parametrize("H,Nq", SHAPES)
def test_prefix_lengths_over_a_few_tiles_are_taken_whole(H, Nq):
    """Where the prefixes end in the first tile, the launch that joins the parts is half of such a call."""
    blocks = H * -(-Nq // 256)
    for tiles in range(1, 48):
        if blocks <= 256 and _parts_of_four_tiles(blocks, tiles) <= 1:
            assert _scratch(H, Nq, tiles, True) == 0, tiles


def test_shared_tiles_have_a_cost_of_their_own():
    """More than 512 queries per unit read tiles that another launch has decoded: a part's start is dear for what it saves."""
    assert _scratch(12, 600, 7) == 0
    assert _scratch(12, 512, 7) > 0
    assert _scratch(1, 600, 7) > 0


def test_misaligned_scratch_of_calls_that_have_always_been_divided_is_refused():
    """With room for their parts of four tiles; the calls below that were ignored it."""
    at = B.C.c_void_p
    fake, odd = at(0x1000), at(0x1008)               # never dereferenced: the call fails first

    def call(H, Nq, n, room):
        return B.lib().qvg_attn_decode_parts(
            B.C.byref(B.make_params(H, 16, 64, 2)), Nq, fake, n, n, 0, fake, fake, fake, fake, fake, fake, fake, fake, None, None,
            B.C.c_float(0.1), fake, None, None, None, 0, odd, room, None)
    assert call(1, 64, 512, 2 * STATE) == -5 and call(1, 64, 4096, 16 * STATE) == -5
    assert call(64, 200, 512, 64 * 2 * STATE) == -5 and call(65, 1, 640, 65 * 2 * STATE) == -5


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("host_parts") / "host_parts")
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    subprocess.run([hipcc, *qbuild.FLAGS, "--offload-host-only", os.path.join(os.path.dirname(os.path.abspath(__file__)), "host_parts.cpp"),
                    "-x", "none", qbuild.LIB, "-Wl,-rpath," + os.path.dirname(qbuild.LIB), "-o", exe], check=True, stderr=subprocess.DEVNULL)
    text = subprocess.run([exe], check=True, capture_output=True, text=True).stdout
    return dict(line.split(" ", 1) for line in text.splitlines())


@pytest.mark.parametrize("name", ["longer_caches", "what_is_asked_for"])
def test_parts_by_the_scratch_that_is_lent(rules, name):
    assert rules[name] == "ok"
