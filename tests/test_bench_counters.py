"""CPU: the counter table prices a matrix instruction by the one its kernel uses."""
import bench


def test_flops_of_a_matrix_instruction():
    bf16, f32 = "unsigned short", "float"
    assert bench.mfma_flop(f"void o5::gemm_kk<256, 256, true, o5::EpiLstmCell<{bf16}>, {bf16}>(...)") == 32768
    assert bench.mfma_flop(f"void o5::step::lstm_step_bwd<{bf16}, 32>(...)") == 32768
    assert bench.mfma_flop(f"void o5::step::lstm_step_fwd<{f32}, 64>(...)") == 2048
    assert bench.mfma_flop(f"void o5::gemm_f32_mfma<128, true, o5::ICols2<{f32}>, o5::ICols2<{f32}>>(...)") == 4096
