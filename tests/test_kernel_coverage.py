"""Every kernel instantiation compiled into libsparrow.so and the GPU test that runs it against the
oracle.  The table below is checked two ways on the CPU: its keys must be exactly the set of
`__global__` instantiations the library holds (read from the library's host stubs, so a new
template instance cannot appear without a line here), and every test it names must exist.  That
every instantiation runs in the test file named for it was observed with a kernel trace of all GPU test
files (profiles/gpu_test_suite_kernel_coverage.txt).

instantiation                                   test file : test (parameters)
"""
import os
import re
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_2602_15318_amd", "libsparrow.so")

A, AC, AS, ASQ, T, H, C, G = ("test_gpu_parity_attn.py", "test_gpu_parity_accept.py",
                              "test_gpu_parity_accept_sample.py", "test_gpu_parity_accept_sample_q.py",
                              "test_gpu_parity_tree.py", "test_gpu_parity_hsr.py",
                              "test_gpu_parity_commit.py", "test_gpu_graph_and_passes.py")

VF, TS = "test_gpu_verify_f32.py", "test_gpu_tree_sizes.py"
V64, LM, HW = "test_gpu_verify_heads64.py", "test_gpu_lm_head_widths.py", "test_gpu_draft_input_widths.py"
VP, VL = "test_gpu_verify_plain_alu.py", "test_gpu_verify_long_trees.py"
DW, VC, VM = "test_gpu_draft_windows.py", "test_gpu_verify_few_splits.py", "test_gpu_verify_long_splits.py"

COVERAGE = {
    # ---- verification attention, matrix cores, bf16: <head_dim, steps in flight, row tiles, streams half a step apart>
    "verify_partial_mfma_kernel<128, 1, 1, false>": (A, "test_c5_bf16_26k_chain8_layer", "C5 layer, C2; chains up to 64 rows per KV head"),
    "verify_partial_mfma_kernel<128, 2, 1, false>": (A, "test_c4_bf16_ragged_batch8", "splits of four steps and more: ragged batch"),
    "verify_partial_mfma_kernel<128, 1, 2, false>": (A, "test_paper_sized_trees_at_26k_context", "16-node tree: one block of 128 rows, short splits"),
    "verify_partial_mfma_kernel<128, 2, 2, true>": (A, "test_c3_bf16_26k_tree60", "C3 60-node tree: several blocks of 128 rows, long splits"),
    "verify_partial_mfma_kernel<128, 2, 2, false>": (VL, "test_split_ends", "one block of 128 rows over long splits; several over shorter ones"),
    "verify_partial_mfma_kernel<128, 1, 3, false>": (A, "test_paper_sized_trees_at_26k_context", "48-, 44- and 25-node trees: blocks of 192 rows"),
    "verify_combine_tiled_kernel<unsigned short, 128, 4>": (A, "test_c3_bf16_26k_tree60", "9 to 16 splits of several row blocks (C3)"),
    "verify_partial_mfma_kernel<64, 1, 0, false>": (V64, "test_rows_of_two_wavefronts", "up to 32 rows"),
    "verify_partial_mfma_kernel<64, 1, 1, false>": (V64, "test_rows_and_contexts", "up to 64 rows, short contexts"),
    "verify_partial_mfma_kernel<64, 2, 1, false>": (V64, "test_batches_and_long_contexts", "26k chain, ragged batch"),
    "verify_partial_mfma_kernel<64, 1, 2, false>": (V64, "test_rows_and_contexts", "70, 240 and 480 rows"),
    "verify_partial_mfma_kernel<64, 2, 2, false>": (V64, "test_two_row_tiles_over_long_pieces", "60 nodes at 26k, 12 trees of 30 at 4k"),
    "verify_partial_mfma_kernel<64, 1, 3, false>": (V64, "test_rows_and_contexts", "175 rows"),
    "verify_combine_tiled_kernel<unsigned short, 64, 4>": (V64, "test_rows_and_contexts", "short contexts"),
    # fp32: <head_dim, row tiles>, <storage type, head_dim, wavefronts>
    "verify_partial_f32_kernel<64, 1>": (VF, "test_rows_and_contexts", "up to 64 rows"),
    "verify_partial_f32_kernel<64, 2>": (VF, "test_rows_and_contexts", "more than 64 rows"),
    "verify_combine_tiled_kernel<float, 64, 4>": (VM, "test_many_splits", "9 to 16 splits of many row blocks"),
    "verify_partial_f32_kernel<128, 1>": (VF, "test_rows_and_contexts", "up to 64 rows"),
    "verify_partial_f32_kernel<128, 2>": (VF, "test_rows_and_contexts", "more than 64 rows"),
    "verify_combine_tiled_kernel<float, 128, 4>": (VM, "test_many_splits", "9 to 16 splits of many row blocks"),
    # merged 16 splits a wavefront: <storage type, head_dim, wavefronts>
    "verify_combine_long_kernel<unsigned short, 64, 1>": (VM, "test_many_splits", "9 to 16 splits, few row blocks"),
    "verify_combine_long_kernel<unsigned short, 64, 2>": (VM, "test_many_splits", "17 to 32 splits"),
    "verify_combine_long_kernel<unsigned short, 64, 4>": (VM, "test_many_splits", "up to 64"),
    "verify_combine_long_kernel<unsigned short, 64, 8>": (VM, "test_many_splits", "up to 128"),
    "verify_combine_long_kernel<unsigned short, 64, 16>": (VM, "test_many_splits", "more"),
    "verify_combine_long_kernel<unsigned short, 128, 1>": (VM, "test_many_splits", "9 to 16 splits, few row blocks"),
    "verify_combine_long_kernel<unsigned short, 128, 2>": (VM, "test_many_splits", "17 to 32 splits"),
    "verify_combine_long_kernel<unsigned short, 128, 4>": (VM, "test_many_splits", "up to 64"),
    "verify_combine_long_kernel<unsigned short, 128, 8>": (VM, "test_many_splits", "up to 128"),
    "verify_combine_long_kernel<unsigned short, 128, 16>": (VM, "test_many_splits", "more"),
    "verify_combine_long_kernel<float, 64, 1>": (VM, "test_many_splits", "9 to 16 splits, few row blocks"),
    "verify_combine_long_kernel<float, 64, 2>": (VM, "test_many_splits", "17 to 32 splits"),
    "verify_combine_long_kernel<float, 64, 4>": (VM, "test_many_splits", "up to 64"),
    "verify_combine_long_kernel<float, 64, 8>": (VM, "test_many_splits", "up to 128"),
    "verify_combine_long_kernel<float, 64, 16>": (VM, "test_many_splits", "more"),
    "verify_combine_long_kernel<float, 128, 1>": (VM, "test_many_splits", "9 to 16 splits, few row blocks"),
    "verify_combine_long_kernel<float, 128, 2>": (VM, "test_many_splits", "17 to 32 splits"),
    "verify_combine_long_kernel<float, 128, 4>": (VM, "test_many_splits", "up to 64"),
    "verify_combine_long_kernel<float, 128, 8>": (VM, "test_many_splits", "up to 128"),
    "verify_combine_long_kernel<float, 128, 16>": (VM, "test_many_splits", "more"),
    # ---- verification attention, plain ALU: <storage type, head_dim>
    # at most 8 and 4 splits per sequence
    "verify_combine_few_kernel<unsigned short, 128, 2>": (VC, "test_few_splits", ""),
    "verify_combine_few_kernel<unsigned short, 128, 1>": (VC, "test_few_splits", ""),
    "verify_combine_few_kernel<unsigned short, 64, 2>": (VC, "test_few_splits", ""),
    "verify_combine_few_kernel<unsigned short, 64, 1>": (VC, "test_few_splits", ""),
    "verify_combine_few_kernel<float, 128, 2>": (VC, "test_few_splits", ""),
    "verify_combine_few_kernel<float, 128, 1>": (VC, "test_few_splits", ""),
    "verify_combine_few_kernel<float, 64, 2>": (VC, "test_few_splits", ""),
    "verify_combine_few_kernel<float, 64, 1>": (VC, "test_few_splits", ""),
    "verify_partial_generic_kernel<float, 64>": (VP, "test_trees_batches_and_splits", "K/V span of 2 GiB"),
    "verify_combine_kernel<float, 64>": (VP, "test_trees_batches_and_splits", "K/V span of 2 GiB"),
    "verify_partial_generic_kernel<float, 128>": (VP, "test_trees_batches_and_splits", "K/V span of 2 GiB"),
    "verify_combine_kernel<float, 128>": (VP, "test_trees_batches_and_splits", "K/V span of 2 GiB"),
    "verify_partial_generic_kernel<unsigned short, 64>": (VP, "test_trees_batches_and_splits", "K/V span of 2 GiB"),
    "verify_combine_kernel<unsigned short, 64>": (VP, "test_trees_batches_and_splits", "K/V span of 2 GiB"),
    "verify_partial_generic_kernel<unsigned short, 128>": (A, "test_kv_span_of_2_gib_takes_the_plain_alu_kernels", "K/V span of 2 GiB"),
    "verify_combine_kernel<unsigned short, 128>": (A, "test_kv_span_of_2_gib_takes_the_plain_alu_kernels", "K/V span of 2 GiB"),
    # ---- draft window attention: <storage type, head_dim>
    # <storage type, head size, workgroups per head, tokens of a round>
    "draft_window_attn_kernel<float, 64, 1, 2>": (DW, "test_shares_and_rounds", ""),
    "draft_window_attn_kernel<float, 64, 1, 8>": (DW, "test_shares_and_rounds", ""),
    "draft_window_attn_kernel<float, 64, 2, 2>": (DW, "test_shares_and_rounds", ""),
    "draft_window_attn_kernel<float, 64, 2, 8>": (DW, "test_shares_and_rounds", ""),
    "draft_window_attn_kernel<float, 64, 4, 2>": (DW, "test_shares_and_rounds", ""),
    "draft_window_attn_kernel<float, 64, 4, 8>": (DW, "test_shares_and_rounds", ""),
    "draft_window_attn_kernel<float, 128, 1, 2>": (DW, "test_shares_and_rounds", ""),
    "draft_window_attn_kernel<float, 128, 1, 8>": (DW, "test_shares_and_rounds", ""),
    "draft_window_attn_kernel<float, 128, 2, 2>": (DW, "test_shares_and_rounds", ""),
    "draft_window_attn_kernel<float, 128, 2, 8>": (DW, "test_shares_and_rounds", ""),
    "draft_window_attn_kernel<float, 128, 4, 2>": (DW, "test_shares_and_rounds", ""),
    "draft_window_attn_kernel<float, 128, 4, 8>": (DW, "test_shares_and_rounds", ""),
    "draft_window_attn_kernel<unsigned short, 64, 1, 2>": (DW, "test_shares_and_rounds", ""),
    "draft_window_attn_kernel<unsigned short, 64, 1, 8>": (DW, "test_shares_and_rounds", ""),
    "draft_window_attn_kernel<unsigned short, 64, 2, 2>": (DW, "test_shares_and_rounds", ""),
    "draft_window_attn_kernel<unsigned short, 64, 2, 8>": (DW, "test_shares_and_rounds", ""),
    "draft_window_attn_kernel<unsigned short, 64, 4, 2>": (DW, "test_shares_and_rounds", ""),
    "draft_window_attn_kernel<unsigned short, 64, 4, 8>": (DW, "test_shares_and_rounds", ""),
    "draft_window_attn_kernel<unsigned short, 128, 1, 2>": (DW, "test_shares_and_rounds", ""),
    "draft_window_attn_kernel<unsigned short, 128, 1, 8>": (DW, "test_shares_and_rounds", ""),
    "draft_window_attn_kernel<unsigned short, 128, 2, 2>": (DW, "test_shares_and_rounds", ""),
    "draft_window_attn_kernel<unsigned short, 128, 2, 8>": (DW, "test_shares_and_rounds", ""),
    "draft_window_attn_kernel<unsigned short, 128, 4, 2>": (DW, "test_shares_and_rounds", ""),
    "draft_window_attn_kernel<unsigned short, 128, 4, 8>": (DW, "test_shares_and_rounds", ""),
    # ---- lm_head + argmax + acceptance
    "lm_head_generic_kernel<float>": (LM, "test_wider_than_the_matrix_core_kernels", "hidden above 2^20"),
    "lm_head_generic_kernel<unsigned short>": (LM, "test_wider_than_the_matrix_core_kernels", "hidden above 8,192"),
    # <slices per wavefront, blocks of 16 rows>
    "lm_head_ksplit_kernel<1, 1>": (AC, "test_c5_full_vocab_accept", "at most 16 rows"),
    "lm_head_ksplit_kernel<1, 2>": (AC, "test_accept_shapes", "bf16-1024-9000-4-7: 17-32 rows"),
    "lm_head_ksplit_kernel<2, 1>": (LM, "test_hidden_sizes", "hidden above 4,096"),
    # <storage type, vocabulary rows and hidden rows of a tile, wavefronts, of these along the vocabulary, bytes of a row per step>
    "lm_head_tiled_kernel<float, 64, 16, 4, 4, 256>": (LM, "test_fp32", "fp32, up to 16 rows"),
    "lm_head_tiled_kernel<float, 128, 16, 4, 4, 256>": (LM, "test_tiles_of_128_vocabulary_rows", "fp32, up to 16 rows"),
    "lm_head_tiled_kernel<float, 64, 32, 4, 4, 256>": (LM, "test_fp32", "fp32, up to 32 rows"),
    "lm_head_tiled_kernel<float, 128, 32, 4, 4, 256>": (LM, "test_tiles_of_128_vocabulary_rows", "fp32, up to 32 rows"),
    "lm_head_tiled_kernel<float, 64, 64, 4, 2, 128>": (LM, "test_fp32", "fp32, up to 64 rows"),
    "lm_head_tiled_kernel<float, 128, 64, 4, 2, 128>": (LM, "test_tiles_of_128_vocabulary_rows", "fp32, up to 64 rows"),
    "lm_head_tiled_kernel<float, 64, 128, 4, 2, 128>": (LM, "test_fp32", "fp32, up to 128 rows"),
    "lm_head_tiled_kernel<float, 128, 128, 4, 2, 128>": (LM, "test_tiles_of_128_vocabulary_rows", "fp32, up to 128 rows"),
    "lm_head_tiled_kernel<unsigned short, 64, 64, 8, 2, 128>": (LM, "test_hidden_sizes", "bf16, up to 64 rows"),
    "lm_head_tiled_kernel<unsigned short, 128, 64, 8, 2, 128>": (LM, "test_whole_vocabularies", "bf16, up to 64 rows"),
    "lm_head_tiled_kernel<unsigned short, 64, 128, 8, 2, 128>": (LM, "test_many_rows", "bf16, up to 128 rows"),
    "lm_head_tiled_kernel<unsigned short, 128, 128, 8, 2, 128>": (LM, "test_tiles_of_128_vocabulary_rows", "bf16, up to 128 rows"),
    "lm_head_tiled_kernel<unsigned short, 64, 256, 8, 2, 128>": (LM, "test_many_rows", "bf16, up to 256 rows"),
    "lm_head_tiled_kernel<unsigned short, 128, 256, 8, 2, 128>": (LM, "test_tiles_of_128_vocabulary_rows", "bf16, up to 256 rows"),
    "accept_finalize_kernel": (AC, "test_accept_shapes", "every greedy case"),
    # <wavefronts of a chunk>
    "logit_stats_kernel<1>": (AS, "test_accept_sample_matches_oracle", "up to four blocks of 256 tokens a chunk, or 16 and 32 rows"),
    "logit_stats_kernel<4>": (AS, "test_vocabularies", "longer chunks"),
    "accept_sample_kernel": (AS, "test_accept_sample_matches_oracle", "deterministic children"),
    # <0: all, 1: up to the first residual's sums, 2: from there>
    "accept_sample_q_kernel<0>": (ASQ, "test_accept_sample_q_matches_oracle", "sampled draft, up to 32,768 tokens"),
    "accept_sample_q_kernel<1>": (ASQ, "test_vocabularies", "above"),
    "residual_sums_kernel": (ASQ, "test_vocabularies", "above"),
    "accept_sample_q_kernel<2>": (ASQ, "test_residuals_of_siblings_over_a_large_vocabulary", "above"),
    # ---- dynamic draft tree
    # <logits a thread owns>
    "topk_chunk_kernel<1>": (T, "test_draft_topk", "vocabularies up to 16,384"),
    "topk_chunk_kernel<4>": (TS, "test_topk_vocabularies", "up to 65,536"),
    "topk_chunk_kernel<10>": (TS, "test_topk_vocabularies", "up to 163,840"),
    "topk_chunk_kernel<16>": (TS, "test_topk_vocabularies", "up to 262,144"),
    "topk_merge_kernel": (T, "test_draft_topk", ""),
    "tree_expand_kernel": (T, "test_tree_expand_and_select", ""),
    "tree_select_kernel<4>": (TS, "test_selection_sizes", "pools above 128"),
    "tree_select_kernel<32>": (TS, "test_selection_sizes", "pools above 256"),
    "tree_select_small_kernel": (T, "test_tree_expand_and_select", "pools up to 128"),
    # ---- draft input and post-accept commit
    "hsr_fc_generic_kernel<float>": (H, "test_hsr_fc", "f32-4-1-64-256"),
    "hsr_fc_mfma_kernel<7, 2>": (H, "test_hsr_fc", "bf16-28-4-128-3584"),
    "hsr_fc_mfma_kernel<8, 2>": (H, "test_hsr_fc", "bf16-32-8-128-4096"),
    "hsr_fc_gemv_kernel<14>": (H, "test_hsr_fc", "bf16-28-4-128-3584, one row"),
    "hsr_fc_gemv_kernel<16>": (H, "test_hsr_fc", "bf16-32-8-128-4096, one row"),
    "draft_qkv_generic_kernel<float>": (H, "test_draft_qkv_append", "f32-4-1-64-256"),
    "draft_qkv_mfma_kernel<7, 1>": (H, "test_draft_qkv_append", "bf16-28-4-128-3584"),
    "draft_qkv_mfma_kernel<8, 1>": (H, "test_draft_qkv_append", "bf16-32-8-128-4096"),
    # hidden sizes other than 3,584 and 4,096; one row: <slices of a weight row in flight>
    "hsr_fc_any_kernel": (HW, "test_hsr_fc", "nine rows and more, five above 3,072"),
    # <rows, slices in flight>
    "hsr_fc_few_kernel<2, 4>": (HW, "test_hsr_fc", "two rows, hidden up to 1,024"),
    "hsr_fc_few_kernel<4, 4>": (HW, "test_hsr_fc_of_few_rows", "three and four rows, hidden up to 1,024"),
    "hsr_fc_few_kernel<2, 10>": (HW, "test_hsr_fc", "two rows"),
    "hsr_fc_few_kernel<4, 10>": (HW, "test_hsr_fc_of_few_rows", "three and four rows"),
    # <at most eight rows>
    "draft_qkv_any_kernel<true>": (HW, "test_draft_qkv_append", "two to eight rows above 4,096 columns"),
    "draft_qkv_once_kernel": (HW, "test_one_slice_a_wavefront", "two to eight rows (from three up to 1,024 columns)"),
    "hsr_fc_once_kernel": (HW, "test_one_slice_a_wavefront", "five to eight rows, hidden up to 3,072"),
    "draft_qkv_any_kernel<false>": (HW, "test_draft_qkv_append", "more"),
    "hsr_fc_any_gemv_kernel<4>": (HW, "test_hsr_fc", "hidden up to 1,024"),
    "hsr_fc_any_gemv_kernel<8>": (HW, "test_hsr_fc", "hidden 1,280"),
    "hsr_fc_any_gemv_kernel<16>": (HW, "test_hsr_fc", "hidden 2,560 and more"),
    "draft_qkv_gemv_kernel<1>": (HW, "test_draft_qkv_append", "one row: hidden up to 512"),
    "draft_qkv_gemv_kernel<4>": (HW, "test_draft_qkv_append", "hidden 1,000, one and two rows"),
    "draft_qkv_gemv_kernel<7>": (HW, "test_draft_qkv_of_one_row_at_whole_slices", "hidden 2,056 to 3,584"),
    "draft_qkv_gemv_kernel<8>": (HW, "test_draft_qkv_append", "hidden 4,104 and more, in two chunks"),
    "kv_commit_kernel": (C, "test_kv_commit_bit_exact", ""),
    # ---- measurement aid (no part of the method, nothing to compare): run, input left alone
    "stream_read_kernel<2>": (G, "test_stream_read_shapes_run", ""),
    "stream_read_kernel<4>": (G, "test_stream_read_shapes_run", ""),
    "stream_read_kernel<8>": (G, "test_stream_read_shapes_run", ""),
    "stream_read_kernel<16>": (G, "test_stream_read_shapes_run", ""),
}


def _compiled_instantiations():
    if not os.path.exists(LIB):
        from paper_2602_15318_amd import build
        build.build()
    out = subprocess.run(["nm", "-C", LIB], capture_output=True, text=True, check=True).stdout
    names = set()
    for line in out.splitlines():
        m = re.search(r"__device_stub__(.*?)\(", line)
        if m:
            names.add(m.group(1))
    return names


def test_every_compiled_kernel_instantiation_has_a_test():
    compiled = _compiled_instantiations()
    assert len(compiled) >= 40, "could not read the kernel list from the library"
    assert compiled == set(COVERAGE), (
        f"not in the table: {sorted(compiled - set(COVERAGE))}; in the table but not compiled: "
        f"{sorted(set(COVERAGE) - compiled)}")


def test_the_named_tests_exist():
    for kernel, (fname, test, _) in COVERAGE.items():
        src = open(os.path.join(ROOT, "tests", fname)).read()
        assert re.search(rf"^def {test}\(", src, flags=re.M), f"{kernel}: {fname} has no {test}"
