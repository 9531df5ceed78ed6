"""A kernel variant's number is part of the interface: programs store it in
configurations (gp_batch_config) and GP2D_VARIANT values.  The numbers below
have been given out and stay with kernels of the same name."""
import paper_1601_00221_amd as gp

GIVEN_OUT = """
k_core_8_6_8_40 k_core_8_6_8_128 k_core_8_8_8_40 k_core_4_8_8_40 k_core_4_8_16_40 k_core_4_12_32_40 k_core_8_8_8_128
k_core_4_8_16_128 k_core_4_12_32_80 k_core_4_8_8_64 k_core_4_8_8_96 k_core_4_8_16_64 k_core_8_6_8_40_a k_core_8_8_8_40_a
k_core_4_8_16_40_a k_core_4_12_32_40_a k_core_8_6_8_56_at k_core_8_8_8_40_at k_core_4_8_16_48_at k_core_4_8_44_48_t
k_core_8_6_20_48_b k_core_8_8_20_32_b k_core_4_12_32_40_b k_core_4_20_32_40 k_core_4_12_44_32_t k_core_4_16_32_40_b
k_core_4_6_20_24_b k_core_4_8_12_48_at k_core_4_8_16_32_a
""".split()


def test_numbers_given_out_keep_their_kernels():
    names = [v["kernel"] for v in gp.variants()]
    assert names[:len(GIVEN_OUT)] == GIVEN_OUT
    assert len(set(names)) == len(names)
