"""The hazard check along every path of a kernel: results of an MFMA behind a branch, a barrier or a loop's edge, operands written in front of one, and
asm LDS reads that a branch would leave in flight; on hand-written listings.  (The compiled kernels are checked with the other rules.)"""
import isa_check

MFMA = "v_mfma_f32_32x32x16_bf16 v[0:15], v[16:19], v[20:23], v[0:15]"
COPY = "v_mov_b32_e32 v40, v3"
ENTRY = "kernel"


def rules(text):
    blocks = isa_check.kernel_blocks("\nkernel:\n" + text + "\n.Lfunc_end0:", ENTRY)
    return [f[0] for f in isa_check.flow_hazards(blocks)]


def test_a_copy_behind_a_barrier_or_a_branch():
    assert rules(f"{MFMA}\ns_barrier\n{COPY}\ns_endpgm") == ["result"]
    assert rules(f"{MFMA}\ns_cbranch_scc1 .LBB0_1\ns_nop 15\n.LBB0_1:\n{COPY}\ns_endpgm") == ["result"]   # if it is taken
    assert rules(f"{MFMA}\ns_branch .LBB0_1\n{COPY}\n.LBB0_1:\ns_nop 15\n{COPY}\ns_endpgm") == []         # the copy in between is not on the way
    assert rules(f"{MFMA}\ns_barrier\ns_nop 10\n{COPY}\ns_endpgm") == []                                 # 12 wait states
    assert rules(f"{MFMA}\ns_barrier\ns_nop 9\n{COPY}\ns_endpgm") == ["result"]


def test_a_loop_leads_from_its_end_to_its_beginning():
    loop = ".LBB0_1:\n%s\ns_nop 15\n%s\ns_cbranch_scc1 .LBB0_1\ns_endpgm"
    assert rules(loop % (COPY, MFMA)) == ["result"]
    assert rules(loop % ("v_mov_b32_e32 v40, v41", MFMA)) == []
    assert rules(loop % (MFMA, "v_mov_b32_e32 v20, 0")) == ["operand"]                                   # one wait state, the branch
    assert rules((loop % (MFMA, "v_mov_b32_e32 v20, 0")).replace(MFMA, "s_nop 0\n" + MFMA)) == []


def test_a_result_that_is_an_operand():
    other = "v_mfma_f32_32x32x16_bf16 v[48:63], v[12:15], v[20:23], v[48:63]"
    assert set(rules(f"{MFMA}\n{other}\ns_endpgm")) == {"result as operand"}
    assert rules(f"{MFMA}\n{MFMA}\ns_endpgm") == []


def test_asm_reads_in_flight():
    read = lambda a: f";;#ASMSTART\nds_read_b128 v[{a}:{a + 3}], v60\n;;#ASMEND"
    use = "v_mov_b32_e32 v70, v17"
    branch = "s_cbranch_scc1 .LBB0_1\ns_nop 0\n.LBB0_1:"
    assert rules(f"{read(16)}\n{branch}\n{use}\ns_endpgm") == ["LDS read in flight"]
    assert rules(f"{read(16)}\n{branch}\ns_waitcnt lgkmcnt(0)\n{use}\ns_endpgm") == []
    assert rules(f"{read(16)}\n{read(20)}\n{branch}\ns_waitcnt lgkmcnt(1)\n{use}\ns_endpgm") == []
    assert rules(f"{read(20)}\n{read(16)}\n{branch}\ns_waitcnt lgkmcnt(1)\n{use}\ns_endpgm") == ["LDS read in flight"]
    # a read behind it on one of the paths only: the other one counts
    more = branch.replace("s_nop 0", read(20))
    assert rules(f"{read(16)}\n{more}\ns_waitcnt lgkmcnt(1)\n{use}\ns_endpgm") == ["LDS read in flight"]
    assert rules(f"ds_read_b128 v[16:19], v60\n{branch}\n{use}\ns_endpgm") == []        # the compiler knows its own
