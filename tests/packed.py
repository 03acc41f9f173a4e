"""A packed cache made from given keys, values and queries, and float64 attention over its bytes.

The pools are filled by the library's encoders (whose bytes other tests pin to the oracle); keys and
values are read back from them with the oracle's unpacking and the reconstruction formulas in float64.
"""
import numpy as np
import torch

from oracle import cache_format, polar, values as ovalues

D, G = 128, 128
DEV = "cuda:0"


class Packed:
    """keys, values: per sequence float arrays [L, KV heads, d]; q [sequences, query heads, d]."""

    def __init__(self, keys, values, q, bits=(4, 4), v_bits=16, max_seq_len=None, residual=False):
        import paper_2502_00527_amd as pq

        self.pq, self.bits, self.v_bits = pq, bits, v_bits
        self.lens = [k.shape[0] for k in keys]
        heads = keys[0].shape[1]
        self.layout = pq.Layout(D, bits[0], bits[1], G, heads)
        self.max_seq_len = max_seq_len or max(self.lens)
        counts = [(n + G - 1) // G for n in self.lens]
        total = sum(counts)
        self.table = np.zeros((len(keys), (self.max_seq_len + G - 1) // G), np.int32)
        ub = 2 * (bits[0] + bits[1])
        self.codes = torch.zeros((total, heads, 4, G, ub), dtype=torch.uint8, device=DEV)
        self.params = torch.zeros((total, heads, 64, 2), dtype=torch.float16, device=DEV)
        self.residual = torch.zeros((len(keys), heads, G, D), dtype=torch.float16, device=DEV) if residual else None
        self.v_params = None
        if v_bits == 16:
            self.v_pool = torch.zeros((total, heads, G, D), dtype=torch.float16, device=DEV)
        else:
            self.v_pool = torch.zeros((total, heads, G * v_bits // 16, 16, 16), dtype=torch.uint8, device=DEV)
            self.v_params = torch.zeros((total, heads, G, 2), dtype=torch.float16, device=DEV)
        self.k64, self.v64 = [], []
        at = 0
        for s, (k, v) in enumerate(zip(keys, values)):
            n, L = counts[s], k.shape[0]
            if L == 0:
                self.k64.append(torch.zeros((0, heads, D), dtype=torch.float64))
                self.v64.append(torch.zeros((0, heads, D), dtype=torch.float64))
                continue
            ids = np.arange(at, at + n, dtype=np.int32)
            self.table[s, :n] = ids
            at += n
            dev_ids = torch.from_numpy(ids).to(DEV)
            packed = L // G * G if residual else L
            k_hat = np.zeros((L, heads, D))
            if packed:
                groups = (packed + G - 1) // G
                pq.pq_encode_keys(self.layout, torch.from_numpy(np.ascontiguousarray(k[:packed])).to(DEV), dev_ids[:groups], self.codes, self.params)
                a, c, scale, zero = cache_format.unpack_pages(self.codes[ids[:groups]].cpu().numpy(), self.params[ids[:groups]].cpu().numpy(), packed, *bits)
                k_hat[:packed] = polar.dequant_keys(a, c, scale, zero, bits[1], G)
            if packed < L:
                tail = torch.from_numpy(k[packed:].astype(np.float16))
                self.residual[s, :, : L - packed] = tail.permute(1, 0, 2).to(DEV)
                k_hat[packed:] = tail.double().numpy()
            self.k64.append(torch.from_numpy(k_hat))
            v16 = torch.from_numpy(v.astype(np.float16)).to(DEV)
            if v_bits == 16:
                rows = torch.zeros((n * G, heads, D), dtype=torch.float16, device=DEV)
                rows[:L] = v16
                self.v_pool[dev_ids.long()] = rows.view(n, G, heads, D).permute(0, 2, 1, 3)
                self.v64.append(v16.double().cpu())
            else:
                pq.pq_encode_values(self.layout, v_bits, v16, dev_ids, self.v_pool, self.v_params)
                codes = cache_format.unpack_value_pages(self.v_pool[ids].cpu().numpy(), L, v_bits)
                par = self.v_params[ids].cpu().numpy().transpose(0, 2, 1, 3).reshape(n * G, heads, 2)[:L]
                self.v64.append(torch.from_numpy(ovalues.dequant_values(codes, par[..., 0], par[..., 1])).double())
        self.q = torch.from_numpy(np.ascontiguousarray(q)).to(DEV)
        self.block_table = torch.from_numpy(self.table).to(DEV)
        self.seq_lens = torch.tensor(self.lens, dtype=torch.int32, device=DEV)
        self.sm_scale = 1.0 / np.sqrt(D)

    def attention(self, scores=None):
        pq, (seqs, heads) = self.pq, self.q.shape[:2]
        out = torch.full((seqs, heads, D), float("nan"), device=DEV)
        size = pq.pq_decode_workspace_bytes(self.layout, seqs, heads, self.max_seq_len)
        guarded = torch.full((size + 4096,), 0x5A, dtype=torch.uint8, device=DEV)
        workspace = guarded[:size]
        pq.pq_decode_attention(self.layout, self.q, self.codes, self.params, self.v_pool, self.block_table, self.seq_lens,
                               self.max_seq_len, self.sm_scale, out, workspace, scores, self.residual, self.v_bits, self.v_params)
        torch.cuda.synchronize()
        assert bool((guarded[size:] == 0x5A).all()), "written past the workspace"
        return out

    def scores(self):
        out = torch.full((*self.q.shape[:2], self.max_seq_len), float("nan"), device=DEV)
        self.pq.pq_score_keys(self.layout, self.q, self.codes, self.params, self.block_table, self.seq_lens, self.max_seq_len, out, self.residual)
        torch.cuda.synchronize()
        return out

    def exact(self):
        """(scores per sequence [query heads, L], attention [sequences, query heads, d]) in float64."""
        all_scores, out = [], []
        for s in range(len(self.lens)):
            k, v = self.k64[s].permute(1, 2, 0).contiguous(), self.v64[s].permute(1, 0, 2).contiguous()      # [H, d, L], [H, L, d]
            q = self.q[s].double().cpu().view(k.shape[0], -1, D)
            scores = torch.matmul(q, k)
            all_scores.append(scores.flatten(0, 1))
            out.append(torch.matmul(torch.softmax(scores * self.sm_scale, dim=-1), v).flatten(0, 1))
        return all_scores, torch.stack(out)


def relative_error(got, want):
    return float((got.double().cpu() - want).norm() / want.norm())
