"""Checks on the generated gfx950 code (no GPU needed): of the FFN kernels for longer blocks, which
use the streaming building block, and of every kernel with matrix instructions.

The kernels for blocks of more than 32 tokens issue their loads from inline asm
and wait for them with explicit counts.  The compiler neither inserts the wait
states the hardware requires around instructions inside asm nor knows that the
loaded registers are valid only after the explicit wait, so three properties
of the generated code are checked here:
  * a scalar register written by a vector instruction (v_readlane /
    v_readfirstlane, e.g. a spilled scalar being restored) is not used as the
    base of a vector-memory load within the next five wait states;
  * the write of M0 and the direct-to-LDS load that uses it are at least one
    wait state apart;
  * those kernels spill no vector registers (a spill could copy a register whose
    asynchronous load has not landed yet);
  * no move, spill or LDS write reads the destination of such a load between the load
    and the explicit wait that covers it (the compiler believes the value is there as
    soon as the asm statement has been issued and could copy it, e.g. on a loop back edge).

Matrix instructions ignore the execution mask.  A block of them under a mask that the compiler
takes for divergent is skipped by a branch only if the compiler thinks the branch worth its
while; without it the block runs with all lanes off and adds what it should not.  So no matrix
instruction may follow a narrowing of the mask that has no branch for "no lane left".
"""
import functools
import os
import re
import tempfile

import pytest

from paper_2602_00879_amd import build as B


@functools.lru_cache(maxsize=None)
def _asm(source):
    with tempfile.TemporaryDirectory() as d:
        return open(B.device_asm(source, os.path.join(d, source + ".s"))).read()


@pytest.fixture(scope="module")
def ffn_asm():
    return _asm("des_ffn.hip")


def _kernels(text):
    """{kernel name: list of instructions} of every kernel in the assembly."""
    out = {}
    for m in re.finditer(r"\n(_ZN3des\w+):[^\n]*\n(.*?)\n\.Lfunc_end", text, re.S):
        ins = []
        for line in m.group(2).split("\n"):
            line = line.split(";")[0].strip()
            if line and not line.startswith(".") and not line.endswith(":"):
                ins.append(line)
        out[m.group(1)] = ins
    return out


def _wait_states(instr):
    m = re.match(r"s_nop (\d+)", instr)
    return int(m.group(1)) + 1 if m else 1


def _scalar_bases(text):
    """{kernel: loads with a scalar base}; none comes less than five wait states after a vector
    instruction that wrote the base."""
    seen = {}
    for name, ins in _kernels(text).items():
        for i, instr in enumerate(ins):
            m = re.match(r"global_load_(?:lds_)?dwordx4 .*s\[(\d+):(\d+)\]", instr)
            if not m:
                continue
            seen[name] = seen.get(name, 0) + 1
            base = {int(m.group(1)), int(m.group(2))}
            ws = 0
            for j in range(i - 1, max(-1, i - 8), -1):
                w = re.match(r"v_(?:readlane|readfirstlane)_b32 s(\d+),", ins[j])
                assert not (w and int(w.group(1)) in base and ws < 5), (
                    f"{name}: '{ins[j]}' only {ws} wait states before '{instr}'")
                ws += _wait_states(ins[j])
    return seen


def _direct_loads(text):
    """{kernel: direct-to-LDS loads}; each comes at least one wait state after the write of M0."""
    seen = {}
    for name, ins in _kernels(text).items():
        for i, instr in enumerate(ins):
            if not instr.startswith("global_load_lds_dwordx4"):
                continue
            seen[name] = seen.get(name, 0) + 1
            j = i - 1
            ws = 0
            while j >= 0 and not ins[j].startswith("s_mov_b32 m0"):
                ws += _wait_states(ins[j])
                j -= 1
                assert i - j < 6, f"{name}: no M0 write just before '{instr}'"
            assert ws >= 1, f"{name}: M0 written immediately before '{instr}'"
    return seen


def test_no_vector_written_scalar_base_too_close_to_a_load(ffn_asm):
    seen = _scalar_bases(ffn_asm)
    assert all(seen.get(k, 0) > 0 for k in _kernels(ffn_asm) if "lds_kernel" in k)


def test_m0_write_is_one_wait_state_before_direct_lds_load(ffn_asm):
    seen = _direct_loads(ffn_asm)
    assert all(seen.get(k, 0) > 0 for k in _kernels(ffn_asm) if "lds_kernel" in k)


def test_asm_load_kernels_do_not_spill(ffn_asm):
    n = 0
    for m in re.finditer(r"\.amdhsa_kernel (\S+)\n(.*?)\.end_amdhsa_kernel", ffn_asm, re.S):
        if "lds_kernel" not in m.group(1):
            continue
        n += 1
        size = int(re.search(r"\.amdhsa_private_segment_fixed_size (\d+)", m.group(2)).group(1))
        assert size == 0, f"{m.group(1)} spills {size} bytes per lane"
    assert n > 0


def test_router_kernels_do_not_spill():
    """Two workgroups of 16 wavefronts share a compute unit: 64 registers each."""
    sizes = {m.group(1): int(m.group(2)) for m in re.finditer(
        r"\.amdhsa_kernel (\S*router_kernel\S*)\n.*?\.amdhsa_private_segment_fixed_size (\d+)", _asm("des_routing.hip"), re.S)}
    assert len(sizes) == 2 and set(sizes.values()) == {0}


def _regs(operand):
    """Vector registers named by one operand: v7 -> {7}, v[4:7] -> {4..7}."""
    m = re.fullmatch(r"v(\d+)", operand)
    if m:
        return {int(m.group(1))}
    m = re.fullmatch(r"v\[(\d+):(\d+)\]", operand)
    if m:
        return set(range(int(m.group(1)), int(m.group(2)) + 1))
    return set()


_TRACKED = [0]  # hand-written loads seen by the scan (the check must not be vacuous)


def _scan_pending_reads(name, ins, pending, errors, prev=""):
    """Walks instructions in text order keeping the vector-memory operations that may
    still be outstanding (they complete in order, so a wait for at most n outstanding
    leaves the last n); an instruction that reads a destination still pending is an error."""
    for instr in ins:
        op, _, rest = instr.partition(" ")
        ops = [o.strip() for o in rest.split(",")] if rest else []
        w = re.search(r"vmcnt\((\d+)\)", instr) if op == "s_waitcnt" else None
        if w:
            n = int(w.group(1))
            pending[:] = pending[-n:] if n > 0 else []
            prev = instr
            continue
        is_vmem = op.startswith(("global_load", "global_store", "global_atomic", "buffer_", "flat_", "scratch_"))
        srcs = ops if op.startswith("global_store") else ops[1:]
        src_regs = set().union(*[_regs(re.sub(r"\s.*", "", o)) for o in srcs]) if srcs else set()
        busy = set().union(*[d for d in pending if d]) if pending else set()
        # what the compiler might do with a value it believes present: copy it (a move at a
        # loop back edge, a move to an accumulation register), spill it or store it.
        # Arithmetic is not flagged: a text-order scan cannot tell that the loop's last
        # trip issued no loads, and the epilogue reuses those registers legitimately.
        copies = op.startswith(("v_mov_b", "v_accvgpr", "v_pk_mov", "scratch_store", "ds_write", "v_swap"))
        if copies and src_regs & busy:
            errors.append(f"{name}: '{instr}' reads v{sorted(src_regs & busy)} before the wait that covers its load")
        if is_vmem:
            # the hand-written loads are the 16-byte non-temporal ones issued right after
            # their own `s_nop 4`; the compiler waits for its own loads itself
            mine = op == "global_load_dwordx4" and instr.endswith(" nt") and prev == "s_nop 4"
            pending.append(_regs(ops[0]) if mine else set())
            _TRACKED[0] += 1 if mine else 0
        prev = instr
    return prev


def test_no_read_of_an_asynchronously_loaded_register_before_its_wait(ffn_asm):
    """Only the loads of the long-block kernels are asynchronous in this sense; their
    kernels are scanned in text order and every loop body (a label followed later by a
    backward branch to it) a second time with the state at the branch, which covers a
    copy on the back edge."""
    errors = []
    n = 0
    _TRACKED[0] = 0
    for m in re.finditer(r"\n(_ZN3des\w*lds_kernel\w+):[^\n]*\n(.*?)\n\.Lfunc_end", ffn_asm, re.S):
        n += 1
        lines = [l.split(";")[0].strip() for l in m.group(2).split("\n")]
        lines = [l for l in lines if l and not l.startswith(".")]
        label_at = {l[:-1]: i for i, l in enumerate(lines) if l.endswith(":")}
        pending = []
        prev = ""
        for i, l in enumerate(lines):
            if l.endswith(":"):
                continue
            prev = _scan_pending_reads(m.group(1), [l], pending, errors, prev)
            b = re.match(r"s_cbranch\w+ (\S+)|s_branch (\S+)", l)
            tgt = (b.group(1) or b.group(2)) if b else None
            if tgt in label_at and label_at[tgt] < i:  # a back edge: once more round the loop
                body = [x for x in lines[label_at[tgt]:i + 1] if not x.endswith(":")]
                _scan_pending_reads(m.group(1), body, list(pending), errors)
    assert n > 0 and _TRACKED[0] > 40
    assert not errors, "\n".join(errors[:10])



def _masked_matrix_instructions(text):
    """(matrix instructions seen, those that run under a narrowed mask without a skip branch)"""
    seen, bad = 0, []
    for m in re.finditer(r"\n(_ZN3des\w+):[^\n]*\n(.*?)\n\.Lfunc_end", text, re.S):
        narrowed = None
        for line in m.group(2).split("\n"):
            ins = line.split(";")[0].strip()
            if re.match(r"s_(and|andn2)_(saveexec_b64|b64 exec, exec)", ins):
                narrowed = ins
            elif re.match(r"s_cbranch_exec|s_(or|mov)_b64 exec|s_or_saveexec", ins):
                narrowed = None
            elif ins.startswith("v_mfma"):
                seen += 1
                if narrowed:
                    bad.append(f"{m.group(1)}: '{ins}' after '{narrowed}'")
    return seen, bad


@pytest.mark.parametrize("source", ["des_ffn.hip", "des_attention.hip", "des_routing.hip"])
def test_no_matrix_instruction_under_a_mask_without_a_skip_branch(source):
    seen, bad = _masked_matrix_instructions(_asm(source))
    assert seen == len(re.findall(r"^\s*v_mfma", _asm(source), re.M)) > 0
    assert not bad, "\n".join(bad[:10])


def test_the_mask_scan_flags_the_pattern():
    mfma = "\tv_mfma_f32_16x16x32_bf16 v[0:3], v[4:7], v[8:11], v[0:3]\n"
    kernel = ("\n_ZN3des1kEv: ; @k\n\ts_and_saveexec_b64 s[0:1], vcc\n%s" + mfma +
              "\ts_or_b64 exec, exec, s[0:1]\n" + mfma + "\ts_endpgm\n.Lfunc_end0:\n")
    seen, bad = _masked_matrix_instructions(kernel % "")
    assert seen == 2 and len(bad) == 1
    assert _masked_matrix_instructions(kernel % "\ts_cbranch_execz .LBB0_2\n") == (2, [])


def test_loads_without_the_non_temporal_hint_are_waited_for_as_well(ffn_asm):
    """The same scan over the hand-written loads of weights that several workgroups read: it knows
    such loads by their hint, so they get one here."""
    hinted, n = re.subn(r"(\ts_nop 4\n\tglobal_load_dwordx4 v\[\d+:\d+\], v\d+, s\[\d+:\d+\](?: offset:\d+)?)[ \t]*(?=\n)",
                        r"\1 nt", ffn_asm)
    assert n > 40
    test_no_read_of_an_asynchronously_loaded_register_before_its_wait(hinted)


def test_direct_lds_loads_of_the_attention_kernels():
    """The two wait-state rules in the file whose projections load both operands straight into LDS, from
    a scalar base, and whose core brings in values so: every such kernel has loads that were looked at."""
    asm = _asm("des_attention.hip")
    bases, direct = _scalar_bases(asm), _direct_loads(asm)
    tiles = [k for k in _kernels(asm) if "linear_tile_kernel" in k]
    straight = [k for k in tiles if not k.split("linear_tile_kernel")[1].startswith("ILi4ELi4ELi1ELi0E")]
    assert len(straight) == len(tiles) - 1 == 9
    for k in straight:
        assert direct.get(k, 0) == bases.get(k, 0) >= 6, k
    rows = [k for k in _kernels(asm) if re.search(r"attention_core_kernelI\w+Lb1E", k)]
    assert len(rows) == 8 and all(direct.get(k, 0) > 0 for k in rows)
    assert set(direct) == set(straight) | set(rows)


def test_packed_gateup_tile_two_chunks_ahead_runs_two_workgroups_per_unit(ffn_asm):
    """Its tiles would fit three times into the 160 KB of a compute unit, which is slower."""
    m = re.search(r"\.amdhsa_kernel (\S*gateup_tile_kernelILb1ELi4ELi2ELi2E\S*)\n(.*?)\.end_amdhsa_kernel", ffn_asm, re.S)
    lds = int(re.search(r"\.amdhsa_group_segment_fixed_size (\d+)", m.group(2)).group(1))
    assert 2 * lds <= 160 * 1024 < 3 * lds
