"""The checks that the build makes on the assembly of the kernels with hand-written waits, on small listings."""
import pytest

from paper_2312_03788_amd import build

MFMA = "\tv_mfma_f32_32x32x16_f16 a[0:15], v[0:3], v[4:7], a[0:15]"
WAIT = "\ts_nop 15"
READS = ["v_accvgpr_read_b32 v9, a3", "v_accvgpr_mov_b32 a20, a3", "ds_write_b128 v9, a[0:3] offset:16", "ds_write_b32 v9, a3",
         "ds_write2_b32 v9, a3, a4 offset1:1", "buffer_store_dwordx2 a[2:3], v9, s[0:3], 0 offen", "flat_store_dword v[10:11], a3",
         "global_store_dword v[10:11], a3, off", "scratch_store_dword off, a3, off", "v_add_f32 v9, v8, a3 ; 4-byte"]


def _check(tmp_path, lines, name="_Z6kernelv"):
    f = tmp_path / "k.s"
    f.write_text("\n".join([name + ":", "; %bb.0:"] + lines + ["\ts_endpgm"]) + "\n")
    build._check_results_behind_wait("k.hip", str(f), "kernel")


@pytest.mark.parametrize("read", READS)
def test_matrix_result_read_too_early_is_found(tmp_path, read):
    """Any use of an accumulator register between an MFMA and two full waits fails the build: copies, LDS writes and every kind of
    store, straight behind the MFMA, behind one wait, and behind two waits with something between them."""
    read = "\t" + read
    for lines in ([MFMA, read], [MFMA, WAIT, read], [MFMA, WAIT, "\tv_mov_b32_e32 v1, 0", WAIT, read], [MFMA, WAIT, WAIT, MFMA, read],
                  [MFMA, "\ts_nop 1", "\ts_nop 15", read]):
        with pytest.raises(RuntimeError, match="too early"):
            _check(tmp_path, lines)


@pytest.mark.parametrize("read", READS)
def test_matrix_result_read_behind_the_wait_passes(tmp_path, read):
    read = "\t" + read
    _check(tmp_path, [read, MFMA, "\tds_read_b128 v[4:7], v9", "\ts_cbranch_scc1 .LBB0_1", ".LBB0_1:", MFMA, WAIT, "\t;;#ASMEND", WAIT, read])
    _check(tmp_path, [MFMA, read], name="_Z5otherv")       # (kernels that the compiler's own wait states serve)
