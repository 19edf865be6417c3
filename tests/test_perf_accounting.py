"""The operations that the reported rates are divided by are the ones that are done."""
import itertools

from paper_2501_16385_amd import perf


def test_symmetric_products_count_one_triangle():
    K, T, N, r = 6, 10, 7, 8
    pairs = len(list(itertools.combinations_with_replacement(range(K), 2)))      # sums of X^T X, or of Delta^T Delta, that differ
    flops = perf.train_flops(N, K, r, T)
    assert flops["gram"] == 2 * pairs * T
    assert flops["loss"] == 2 * pairs * N
    # B A, B^T Delta, [Q; At] H, Delta V: N x K x r, r x K x N, 2 r x K x K and N x r x K multiply-adds
    assert flops["step"] == 2 * (N * K * r + r * K * N + 2 * r * K * K + N * r * K)
