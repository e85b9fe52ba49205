"""Sizes of the training workspace (host code only)."""
import paper_1905_13746_amd as nbg


def test_training_workspace_never_shrinks_with_more_files():
    """A workspace for n files serves every smaller call."""
    lib = nbg.load()
    for C, F, x in ((2, 200, 0), (2, 1000, 1), (3, 64, 0), (7, 500, 1), (16, 4096, 0), (40, 1000, 0)):
        last = 0
        for n in sorted({int(1.17 ** i) for i in range(90)} | {48 * 4096 - 1, 48 * 4096, 48 * 4096 + 1, 200_003}):
            size = lib.nb_train_workspace_bytes(C, F, n, x)
            assert size >= last, (C, F, x, n)
            last = size
