"""An idx_allocator over torch tensors that counts the library's requests and
can refuse large ones, indexes built through it, and exact expected answers."""
import ctypes

import torch

import paper_2506_01576_amd as idx


class Arena:
    """Refuses requests above `limit`; `asked` lists the granted sizes."""

    def __init__(self):
        self.limit, self.blocks, self.refused, self.asked = 1 << 62, {}, 0, []
        fields = dict(idx.idx_allocator._fields_)
        self.c = idx.idx_allocator(fields["alloc"](self._alloc), fields["release"](self._release), None)

    def _alloc(self, ctx, nbytes, stream):
        if nbytes > self.limit:
            self.refused += 1
            return None
        self.asked.append(nbytes)
        t = torch.empty(nbytes, dtype=torch.uint8, device="cuda")
        self.blocks[t.data_ptr()] = t
        return t.data_ptr()

    def _release(self, ctx, p, stream):
        torch.cuda.synchronize()
        del self.blocks[p]

    def index(self, keys, rows, layout, k=1, aos=False):
        flags = (idx.IDX_KEY_U64 if keys.element_size() == 8 else 0) | (
            idx.IDX_AOS | idx.IDX_AOS_PADDED if aos == "padded" else idx.IDX_AOS if aos else 0)
        lay = {"bs": idx.IDX_BS, "ebs": idx.IDX_EBS, "eks": idx.IDX_EKS}[layout]
        k = {"bs": 1, "ebs": 2, "eks": k}[layout]
        h = ctypes.c_void_p()
        st = idx.lib().idx_build(keys.data_ptr(), rows.data_ptr(), len(keys), lay, k, flags, ctypes.byref(self.c),
                                 torch.cuda.current_stream().cuda_stream, ctypes.byref(h))
        assert st == idx.IDX_OK, st
        return idx.Index._wrap(h, len(keys), k, layout, 8 * keys.element_size(), keys.dtype)


def ordered(keys):
    """int64 values in the unsigned order of the keys' bits."""
    if keys.element_size() == 4:
        return keys.to(torch.int64) & 0xFFFFFFFF
    return keys ^ (-1 << 63)


def expected_points(keys, rows, q):
    """The first row of every queried key in stable order, or the sentinel."""
    sk, perm = torch.sort(ordered(keys), stable=True)
    x = ordered(q)
    at = torch.searchsorted(sk, x).clamp_(max=len(sk) - 1)
    return torch.where(sk[at] == x, rows[perm[at]], torch.full_like(rows[:1], -1))
