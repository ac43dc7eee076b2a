"""The generated code keeps the contract of the assembly loads with register destinations (register-fed row block
of the wide GEMM tile): nothing touches their destination registers between the request and the wait that retires
them; no wave passes a barrier with LDS writes of its own under way;
and no lane mask of a loop decides for the whole wave behind it.  CPU only: the device code is compiled to assembly and read; the checker itself is tried on planted text."""
import os

import pytest

from paper_2605_23764_amd.asm_check import (barrier_violations, check_register_fed_loads, device_assembly, innermost_loops,
                                            loads_ahead_of_first_branch, stale_lane_masks)

GOOD = """
\t.amdhsa_kernel k
k:
\t;;#ASMSTART
\tglobal_load_dwordx4 v[10:13], v166, s[2:3] offset:32
\t;;#ASMEND
\tv_add_u32_e32 v14, v9, v20
\tds_read_b128 v[20:23], v5
\t;;#ASMSTART
\tv_mfma_f32_32x32x16_bf16 v[30:45], v[20:23], v[24:27], v[30:45]
\t;;#ASMEND
\ts_waitcnt vmcnt(8)
\ts_barrier
\t;;#ASMSTART
\ts_waitcnt vmcnt(8)
\t;;#ASMEND
\tv_mov_b32_e32 v50, v10
"""


def test_checker_accepts_a_clean_window_and_names_planted_mistakes():
    assert check_register_fed_loads(GOOD) == (1, [])
    # a copy of a destination register before the naming wait (what the compiler did to a value carried round a loop)
    n, bad = check_register_fed_loads(GOOD.replace("v_add_u32_e32 v14, v9, v20", "v_mov_b32_e32 v60, v12"))
    assert n == 1 and len(bad) == 1 and bad[0][2] == [12]
    # a destination register reused as scratch inside the window
    n, bad = check_register_fed_loads(GOOD.replace("ds_read_b128 v[20:23], v5", "ds_read_b128 v[12:15], v5"))
    assert len(bad) == 1 and bad[0][2] == [12, 13]
    # an MFMA fed from the block before it has been retired
    n, bad = check_register_fed_loads(GOOD.replace("v[20:23], v[24:27]", "v[20:23], v[10:13]"))
    assert len(bad) == 1 and bad[0][2] == [10, 11, 12, 13]
    # the compiler's own wait does not end the window: only the assembly wait that names the registers does
    n, bad = check_register_fed_loads(GOOD.replace("\ts_barrier\n", "\ts_barrier\n\tv_mov_b32_e32 v61, v11\n"))
    assert len(bad) == 1 and bad[0][2] == [11]


LOOP = """
\t.amdhsa_kernel k
k:
\tds_write_b32 v1, v2
\ts_waitcnt lgkmcnt(0)
.LBB0_1:
\ts_barrier
\tds_read_b32 v3, v4
\ts_waitcnt lgkmcnt(0)
\ts_barrier
\ts_cbranch_scc1 .LBB0_3
\tds_or_b32 v1, v2
\tds_read_b32 v3, v4
\ts_waitcnt lgkmcnt(1)
\ts_branch .LBB0_1
.LBB0_3:
\ts_endpgm
.Lfunc_end0:
"""


def test_barrier_checker_follows_the_loop():
    assert barrier_violations(LOOP) == (2, [])
    # outstanding along the way back alone
    n, bad = barrier_violations(LOOP.replace("\ts_waitcnt lgkmcnt(1)\n", ""))
    assert n == 2 and bad == [("k", 7, 12)]
    # on the way in; a wait that is not long enough; a wait for something else
    for plant in (LOOP.replace("v2\n\ts_waitcnt lgkmcnt(0)\n.LBB0_1", "v2\n.LBB0_1"), LOOP.replace("lgkmcnt(1)", "lgkmcnt(2)"),
                  LOOP.replace("lgkmcnt(1)", "vmcnt(0)")):
        assert len(barrier_violations(plant)[1]) == 1, plant
    # the way back as a long branch
    far = LOOP.replace("\ts_branch .LBB0_1", "\ts_add_u32 s8, s8, (.LBB0_1-.Lpost_getpc0)&4294967295\n\ts_setpc_b64 s[8:9]")
    assert barrier_violations(far) == (2, [])
    assert barrier_violations(far.replace("\ts_waitcnt lgkmcnt(1)\n", ""))[1] == [("k", 7, 12)]


@pytest.mark.skipif(not os.path.exists(os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")), reason="needs hipcc")
def test_no_barrier_is_passed_with_lds_writes_under_way():
    n, bad = barrier_violations(device_assembly())
    assert n > 500, n
    assert not bad, bad[:5]


LANES = """
\t.amdhsa_kernel k
k:
\ts_mov_b64 s[6:7], 0
\ts_branch .LBB0_2
.LBB0_1:
\tv_cmp_le_i32_e32 vcc, s8, v1
\ts_or_b64 s[6:7], vcc, s[6:7]
\ts_andn2_b64 exec, exec, s[6:7]
\ts_cbranch_execz .LBB0_4
.LBB0_2:
\tv_cmp_ne_u32_e64 s[4:5], 1, v2
\ts_and_b64 vcc, exec, s[4:5]
\ts_cbranch_vccnz .LBB0_1
\tglobal_store_dword v3, v4, s[2:3]
\ts_branch .LBB0_1
.LBB0_4:
\ts_or_b64 exec, exec, s[6:7]
\ts_andn2_b64 vcc, exec, s[10:11]
\ts_cbranch_vccnz .LBB0_5
\tglobal_store_dword v3, v4, s[2:3]
.LBB0_5:
\ts_endpgm
.Lfunc_end0:
"""


def test_lane_mask_checker_looks_behind_the_loop():
    assert stale_lane_masks(LANES) == (1, [])
    stale = LANES.replace("s_andn2_b64 vcc, exec, s[10:11]", "s_and_b64 vcc, exec, s[4:5]")
    assert stale_lane_masks(stale) == (1, [("k", 19, 12)])
    # the mask is computed again behind the loop; written by something else; its register is not read as a mask of the wave
    for fresh in ("v_cmp_ne_u32_e64 s[4:5], 1, v2", "s_mov_b64 s[4:5], 0"):
        assert stale_lane_masks(stale.replace("\ts_and_b64 vcc, exec, s[4:5]\n\ts_cbranch_vccnz .LBB0_5", f"\t{fresh}\n\ts_and_b64 vcc, exec, s[4:5]\n\ts_cbranch_vccnz .LBB0_5")) == (1, [])
    assert stale_lane_masks(stale.replace("vcc, exec, s[4:5]\n\ts_cbranch_vccnz .LBB0_5", "s[12:13], exec, s[4:5]\n\ts_cbranch_scc1 .LBB0_5"))[1] == []


@pytest.mark.skipif(not os.path.exists(os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")), reason="needs hipcc")
def test_no_lane_mask_of_a_loop_decides_for_the_wave_behind_it():
    n, bad = stale_lane_masks(device_assembly())
    assert n > 100, n
    assert not bad, bad[:5]


@pytest.mark.skipif(not os.path.exists(os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")), reason="needs hipcc")
def test_generated_code_keeps_the_window_closed():
    n, bad = check_register_fed_loads(device_assembly())
    # four fragments per request, two requests (prologue, loop) per instantiation of the register-fed tile
    assert n >= 8 and n % 4 == 0, n
    assert not bad, bad[:5]


@pytest.mark.skipif(not os.path.exists(os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")), reason="needs hipcc")
@pytest.mark.parametrize("lay,epi", [(0, 1), (0, 0), (1, 2), (1, 0)])
def test_launch_head_waits_for_the_tile_map_once(lay, epi):
    """The number of M tiles (word 0) and the rows of the largest expert (word 3), between which the grouped GEMM kernel
    decides what it runs as, are fetched together."""
    groups = loads_ahead_of_first_branch(device_assembly(), f"_ZN3moe24grouped_gemm_bf16_kernelILi{lay}ELi{epi}EEEvNS_10GemmParamsE")
    # kernel arguments come from s[0:1]
    assert any({(base, 0), (base, 12)} <= set(g) for g in groups for base, _ in g if base != "s[0:1]"), groups


@pytest.mark.skipif(not os.path.exists(os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")), reason="needs hipcc")
def test_fp32_single_launch_keeps_the_addresses_of_its_tiles():
    """No address is added up inside the K loops of whole tiles: GEMM-1 (two column blocks, 32 MFMAs per two steps) and GEMM-2."""
    asm = device_assembly()
    loops = innermost_loops(asm, "_ZN3moe25persistent_forward_kernelILb0ELb0EEEvNS_11SchedParamsIXT_EEE")
    tiles = {sum("v_mfma_f32_32x32x2_f32" in i for i in loop): loop for loop in loops}
    for mfmas in (16, 32):
        assert not [i for i in tiles[mfmas] if i.startswith("v_add_u32")], tiles[mfmas]
