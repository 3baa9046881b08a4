"""Results that calls hand back to the host: from several threads and streams at once, and on deep trees of the heuristic."""
import threading

import numpy as np
import pytest

import oracle
from paper_2308_09723_amd import workloads
from gpu_util import torch_mod

pytestmark = pytest.mark.gpu


def test_results_of_calls_from_several_threads_and_streams():
    """Eight threads, each on a stream of its own with a matrix of its own, call the heuristic and the error report in turn:
    every call returns its own result (the place a call's kernels write it to is shared by all threads)."""
    from paper_2308_09723_amd import fq
    torch = torch_mod()
    mats = []
    for i in range(8):
        W = workloads.weights_gaussian(1024, 256 + 16 * i, 30 + i, outlier_prob=0.0)
        if i % 2:
            W[64 * i:64 * i + 64] *= np.float16(16.0)          # a band of wide groups: another group size
        Wd = torch.from_numpy(W).cuda()
        codes, scales = fq.quantize(Wd, 4, 64)
        mats.append((Wd, codes, scales, fq.choose_group(Wd, 0, 32, 0.9), fq.quant_error(Wd, codes, scales, 4, 64)))
    assert len({m[3] for m in mats}) > 1
    torch.cuda.synchronize()
    wrong = []

    def work(i):
        W, codes, scales, g, err = mats[i]
        with torch.cuda.stream(torch.cuda.Stream()):
            for _ in range(40):
                if fq.choose_group(W, 0, 32, 0.9) != g or fq.quant_error(W, codes, scales, 4, 64) != err:
                    wrong.append(i)

    threads = [threading.Thread(target=work, args=(i,)) for i in range(8)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not wrong


@pytest.mark.parametrize("K,N,g_min", [(65536, 48, 32), (32768, 16, 16), (1024, 4112, 32)])
def test_choose_group_flags_of_many_blocks(K, N, g_min):
    """Trees of more than ten levels (one grid layer per level) and few columns; flags set in one block alone."""
    from paper_2308_09723_amd import fq
    torch = torch_mod()
    W = (np.random.default_rng(K + N).standard_normal((K, N)) * 0.02).astype(np.float16)
    for row, col in ((None, None), (K - 1, N - 1), (0, N // 2)):
        X = W.copy()
        if row is not None:
            X[row, col] = 8.0
        for alpha in (0.0, 0.5, 0.99):
            assert fq.choose_group(torch.from_numpy(X).cuda(), 0, g_min, alpha) == oracle.choose_group(X, 0, g_min, alpha), (row, alpha)


@pytest.mark.parametrize("K,N,g_start,g_min", [(8320, 4112, 64, 32), (16640, 48, 128, 32), (2048, 4112, 256, 32), (512, 8208, 512, 32)])
def test_choose_group_items_of_the_halving_tree(K, N, g_start, g_min):
    """1 - 4 halvings below several top groups: more items than blocks, ragged last items; the one group that halves stands anywhere."""
    from paper_2308_09723_amd import fq
    torch = torch_mod()
    W = np.ones((K, N), dtype=np.float16)
    for row, col in ((None, None), (0, 0), (K - 1, N - 1), (K // 2, N // 2 + 5), (K - g_start, 17)):
        X = W.copy()
        if row is not None:
            X[row, col] = 8.0
        for alpha in (0.5, 0.9):
            assert fq.choose_group(torch.from_numpy(X).cuda(), g_start, g_min, alpha) == oracle.choose_group(X, g_start, g_min, alpha), (row, alpha)
    X = (np.random.default_rng(K + N).standard_normal((K, N)) * 0.02).astype(np.float16)
    X[K // 3, 5], X[K // 2, 9], X[1, N - 1] = np.inf, np.nan, -np.inf
    for alpha in (0.2, 0.6, 0.9):
        assert fq.choose_group(torch.from_numpy(X).cuda(), g_start, g_min, alpha) == oracle.choose_group(X, g_start, g_min, alpha), alpha
