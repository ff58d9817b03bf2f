"""The batches the GPU tests of the balanced decomposition run (tests/test_gpu_balanced.py,
tests/test_gpu_work_cut.py),
kept in one place so that a CPU test (tests/test_work_cut.py) can check that each of them
really takes the balanced cut.  Plain Python: lengths and shapes only, no arithmetic of the
method."""
import random

# (workload id, KV heads, sequence lengths): the Llama-8B attention shape (8 KV heads) with six
# sequences of 1.8K-4K tokens, and the Qwen-7B shape (4 KV heads) with twelve of 65-1455 tokens
RAGGED = [(5, 8, [4000, 2500, 3300, 1800, 4096, 2100]),
          (4, 4, [76, 1379, 1267, 696, 1455, 170, 174, 86, 65, 157, 168, 827])]

# (group size, seed) of the seeded random shapes
RANDOM = [(1, 0), (2, 9), (3, 10), (4, 3), (5, 4), (6, 5), (7, 6), (8, 7)]

# batch sizes at the balanced cut's limit (one sequence per lane of a 64-lane wave), on the
# Qwen-1.5B attention shape (2 KV heads)
BATCH_LIMIT = [64, 65]
BATCH_LIMIT_KV_HEADS = 2


def random_case(seed):
    """KV heads, head dim and lengths of the seeded random shape `seed`: 2, 4 or 8 KV heads,
    head dim 64 or 128, 6-24 sequences of lengths in [L/4, L]."""
    r = random.Random(seed)
    hkv = r.choice([2, 4, 8])
    d = r.choice([64, 128])
    B = r.randint(6, 24)
    L = r.randint(600, 3000)
    lens = [r.randint(L // 4, L) for _ in range(B)]
    return hkv, d, lens


def batch_limit_lens(B):
    r = random.Random(B)
    return [r.randint(400, 800) for _ in range(B)]


# sequences so short that a run spans up to three pairs (8 KV heads)
SHORT_PIECES = [1 + 37 * i % 290 for i in range(48)]

# pieces longer than the kernel's list of 1024 pages, listed in parts: (KV heads, lengths, whether
# the balanced cut is taken), one query head per KV head, and the sequence and head pairs to check
LONG_PIECES = [(128, [16401, 17000], False, [(0, 0), (1, 77), (1, 127)]),
               (128, [17000, 33000], True, [(0, 0), (0, 90), (1, 0), (1, 77), (1, 127)])]

# single-token selections (sequences, KV heads, budget, head dim) whose pieces are longer than the
# list's 64 groups of 16 tokens: 128 groups (walked in blocks of four), 86 and 256
LONG_TOKEN_PIECES = [(32, 8, 2048, 64, 128), (20, 8, 4096, 128, 86), (48, 8, 4096, 64, 256)]

# sparse launches at the edges of their split rule (sequences, KV heads, budget, unit, splits): three
# splits just above one pair per CU (96 groups, and one at 95), one pair per CU and one piece less,
# most splits, two pieces per CU for single tokens from 33 to 255 pairs
SPARSE_SPLITS = [(33, 8, 1536, 16, 3), (33, 8, 1520, 16, 1), (32, 8, 512, 16, 1), (43, 3, 512, 16, 1),
                 (1, 1, 4096, 16, 32), (11, 3, 1024, 1, 8), (4, 8, 1024, 1, 8), (51, 5, 512, 1, 2),
                 (64, 4, 512, 1, 1)]
