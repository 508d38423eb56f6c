"""The selection's definition in torch, for the GPU tests that compare bit for bit."""
import torch


def top(v, k):
    """Positions of the k largest magnitudes, lowest positions first among equals, ascending."""
    key = v.view(torch.int32) & 0x7FFFFFFF
    bar = key.topk(k).values[-1]
    above, equal = (key > bar).nonzero()[:, 0], (key == bar).nonzero()[:, 0]
    return torch.cat([above, equal[:k - above.numel()]]).sort().values
