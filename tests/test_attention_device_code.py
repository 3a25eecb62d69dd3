"""What the built device code of the attention forward shows and no run does (no GPU).

Order: the kernel refills the LDS buffer of K tile 0 (with K tile 2) while it works on tile 0.  The logits of
tile 0 are taken before that, from the same buffer, by all four waves, each at its own pace: a workgroup barrier has to
stand between those reads and the first request that refills the buffer, on every path.  Which wave gets there first
depends on timing.

Registers: a spill costs most where a launch is short, and no result shows it."""
import re

import pytest

from paper_2505_05856_amd import build as bld

LABEL = re.compile(r"^(\.LBB\w+):")


def kernels(asm, part):
    """{name: [instruction or label, ...]} of the kernels whose name holds `part`."""
    out, body = {}, None
    for line in asm.splitlines():
        code = line.split(";", 1)[0].strip()
        m = re.match(r"^(_Z\w+):", line)
        if m:
            body = out.setdefault(m.group(1), []) if part in m.group(1) else None
        elif code.startswith(".Lfunc_end"):
            body = None
        elif body is not None and (LABEL.match(code) or (code and code[0] not in ".#")):
            body.append(code)
    return out


def until_next_barrier(body, start):
    """Every instruction some path reaches from index `start` before it meets a barrier or the end."""
    at = {LABEL.match(c).group(1): i for i, c in enumerate(body) if LABEL.match(c)}
    seen, todo = set(), [start]
    while todo:
        i = todo.pop()
        while i < len(body) and i not in seen:
            op, *args = body[i].split()
            if op in ("s_barrier", "s_endpgm"):
                break
            seen.add(i)
            if op.startswith("s_cbranch"):
                todo.append(at[args[0]])
            if op == "s_branch":
                i = at[args[0]]
                continue
            i += 1
    return [body[i] for i in sorted(seen)]


@pytest.fixture(scope="module")
def device_code(tmp_path_factory):
    path = tmp_path_factory.mktemp("asm") / "attn_mfma.s"
    bld.device_asm("attn_mfma.hip", str(path))
    return path.read_text()


def test_tile_0_is_read_by_everyone_before_its_buffer_is_refilled(device_code):
    forward = kernels(device_code, "attn_fwd_mfma_kernel")
    assert len(forward) >= 8      # both head dimensions, causal or not, dropout or not
    for name, body in forward.items():
        first = next(i for i, c in enumerate(body) if c == "s_barrier")     # certifies K tile 0
        part = until_next_barrier(body, first + 1)
        reads = [c for c in part if c.startswith("ds_read_b128")]
        assert len(reads) >= (8 if "ILi64E" in name else 16), name          # the logits of tile 0 are taken here
        assert not [c for c in part if c.startswith("global_load_lds")], name


# kernel template arguments (head dimension, causal, dropout, waves a SIMD) -> bytes of scratch memory a lane.  The form cut
# for three workgroups a CU and causal dropout at head dimension 128 may keep a few registers there.
@pytest.mark.parametrize("dh,wpe,limit", [(64, 2, 0), (64, 3, 32), (128, 2, 16)])
@pytest.mark.parametrize("causal", [0, 1])
@pytest.mark.parametrize("drop", [0, 1])
def test_the_forward_stays_in_its_registers(device_code, dh, wpe, limit, causal, drop):
    sizes = re.findall(rf"\.amdhsa_kernel _Z\w*attn_fwd_mfma_kernelILi{dh}ELb{causal}ELb{drop}ELi{wpe}E\w*\n(?:.*\n)*?"
                       r"\s*\.amdhsa_private_segment_fixed_size (\d+)", device_code)
    assert len(sizes) == 1 + causal      # causal blocks also in an order of their own
    assert max(map(int, sizes)) <= (limit if wpe == 3 or drop else 0)
