"""A Llama-shaped attention layer on the SWAN cache, in the paper's model-side form.

Sec. 4.2: queries and keys take RoPE first and are then rotated by P_QK at run
time (RoPE keeps P_QK out of W_Q and W_K), while P_VO is absorbed into the
weights, W_V_hat = W_V . P_VO per KV head and W_O_hat = P_VO^T . W_O per query
head, so the values enter the cache already rotated and the attention output
leaves it rotated, straight into W_O_hat (Lemma 2).

One call with n new tokens per sequence, on the current stream:
  [q | k | v_hat] = x . [W_Q | W_K | W_V_hat]    one dense GEMM (torch: the GEMM library)
  swan_rope on q and k at each sequence's next positions
  a prompt (n > 1): swan_compress_append(k, v_hat, P_QK, P_VO = NULL)
  a decode step (n = 1): swan_decode_step(k, v_hat, q, P_QK, P_VO = NULL) -> o_hat
  (the append, then the attention, in one call), and
  y = o_hat . W_O_hat                             dense GEMM
The SWAN steps run in libswan's kernels; attention over a prompt is the dense,
standard kind and is not part of this layer (a prompt call only fills the cache).
Weights are [in][out] row-major, x . W.
"""
from __future__ import annotations

from typing import Optional, Sequence

from . import swan

HEAD_DIM = swan.HEAD_DIM

# joint matrices and solver workspaces that calibrate_joint holds at a time: a layer of
# 32 kv heads and 4096 calibration tokens at once (0.49 GB), longer ones a few heads at a time
JOINT_BYTES = 512 << 20


def calibrate_joint(q, k, v, W_o, n_kv_heads: int, P_qk_out, P_vo_out, stream=None) -> None:
    """The layer's rotations from calibration activations (Sec. 4.1.1-4.1.2).

    q [N_q][n][128]: post-RoPE queries of n calibration tokens; k [N_kv][n][128]
    post-RoPE keys; v [N_kv][n][128] values (x . W_V, before any rotation);
    W_o [N_q 128][hidden] (cuda tensors, float16 or float32).  For each KV head j
    (query heads jG .. jG + G - 1) the joint matrices are stacked in device
    memory as float32, S_QK = [Q_grouped^(j); K^(j)] and S_VO = [V^(j); W_O^(h)^T
    for the group's heads], W_O^(h) being rows 128 h .. 128 h + 127 of W_o, and
    swan_calibrate_rotations writes their right singular matrices to P_qk_out[j]
    and P_vo_out[j] ([N_kv][128][128] float32).  The matrices are solved side by side in
    groups of at most JOINT_BYTES, or one at a time where one is larger."""
    import torch

    n_q, n, d = q.shape
    if d != HEAD_DIM or n_q % n_kv_heads != 0:
        raise ValueError("q must be [N_q][n][128] with N_q a multiple of n_kv_heads")
    if tuple(k.shape) != (n_kv_heads, n, d) or tuple(v.shape) != (n_kv_heads, n, d):
        raise ValueError("k and v must be [n_kv_heads][n][128]")
    if W_o.dim() != 2 or W_o.shape[0] != n_q * d:
        raise ValueError("W_o must be [N_q * 128][hidden]")
    for name, out in (("P_qk_out", P_qk_out), ("P_vo_out", P_vo_out)):
        for j in range(n_kv_heads):
            m = out[j]
            if m.dtype != torch.float32 or not m.is_cuda:
                raise ValueError(f"{name}[{j}] must be a [128][128] float32 cuda matrix")
            swan._tensor(m, name, torch.float32, (d, d))
    swan._on_gpu(q=q)
    if any(t.device != q.device for t in (k, v, W_o)):
        raise ValueError(f"q is on {q.device}, k on {k.device}, v on {v.device}, "
                         f"W_o on {W_o.device}: all must be on one GPU")
    G = n_q // n_kv_heads
    hidden = W_o.shape[1]
    on = torch.cuda.current_stream(q.device)
    if stream is not None:  # the inputs may come from either stream
        stream.wait_stream(on)
        on = stream
    # autograd has no part in this: W_o and the outputs may be parameters
    with torch.inference_mode(), torch.cuda.stream(on):
        q_grouped = q.reshape(n_kv_heads, n * G, d)
        wo_t = W_o.reshape(n_kv_heads, G, d, hidden).transpose(2, 3)  # W_O^(h) transposed
        rows_qk, rows_vo = n * (G + 1), n + G * hidden
        # the problems, S_QK of the heads, then S_VO; the first p0 of them are done
        rows = [rows_qk] * n_kv_heads + [rows_vo] * n_kv_heads
        workspace = swan.calibrate_workspace_bytes(d)
        P = torch.empty((2 * n_kv_heads, d, d), dtype=torch.float32, device=q.device)
        p0 = 0
        while p0 < len(rows):
            p1, held = p0, 0  # the group p0 .. p1 - 1, in one array, solved side by side
            while p1 < len(rows):
                held += 4 * d * rows[p1] + workspace
                if held > JOINT_BYTES and p1 > p0:
                    break
                p1 += 1
            s = torch.empty((sum(rows[p0:p1]), d), dtype=torch.float32, device=q.device)
            h0, h1 = min(p0, n_kv_heads), min(p1, n_kv_heads)
            s_qk = s[:(h1 - h0) * rows_qk].view(h1 - h0, rows_qk, d)
            s_qk[:, :n * G] = q_grouped[h0:h1]
            s_qk[:, n * G:] = k[h0:h1]
            g0, g1 = max(p0 - n_kv_heads, 0), max(p1 - n_kv_heads, 0)
            s_vo = s[(h1 - h0) * rows_qk:].view(g1 - g0, rows_vo, d)
            s_vo[:, :n] = v[g0:g1]
            s_vo[:, n:].unflatten(1, (G, hidden)).copy_(wo_t[g0:g1])
            swan.calibrate_rotations(s, rows[p0:p1], P[p0:p1], stream=on)
            del s, s_qk, s_vo  # before the next group's
            p0 = p1
        for out, got in ((P_qk_out, P[:n_kv_heads]), (P_vo_out, P[n_kv_heads:])):
            if isinstance(out, torch.Tensor):
                out[:n_kv_heads].copy_(got.view(out[:n_kv_heads].shape))
            else:  # a list of matrices
                for j in range(n_kv_heads):
                    out[j].copy_(got[j])
    on.synchronize()  # the rotations are in place on return, for any stream


class SwanAttentionLayer:
    def __init__(self, W_q, W_k, W_v, W_o, P_qk, P_vo, n_heads: int, n_kv_heads: int,
                 rope_base: float, batch: int, buffer_tokens: int, capacity: int,
                 k_active: Sequence[int], k_value: Optional[Sequence[int]] = None,
                 sparse_values: str = "same"):
        """W_q [hidden][n_heads*128], W_k and W_v [hidden][n_kv*128], W_o
        [n_heads*128][hidden] (float16 or float32, cuda); P_qk, P_vo [n_kv][128][128]
        float32 (swan_calibrate_rotation of post-RoPE keys and of values)."""
        import torch

        d = HEAD_DIM
        self.n_heads, self.n_kv_heads = n_heads, n_kv_heads
        self.rope_base = float(rope_base)
        self.dtype = W_q.dtype
        self.P_qk = P_qk.contiguous()
        G = n_heads // n_kv_heads
        # absorbed weights, formed once in float64 and rounded to the weights' type
        Wv = W_v.double().clone()
        Wo = W_o.double().clone()
        P = P_vo.double()
        for h in range(n_kv_heads):
            Wv[:, h * d:(h + 1) * d] = Wv[:, h * d:(h + 1) * d] @ P[h]
        for hq in range(n_heads):
            Wo[hq * d:(hq + 1) * d, :] = P[hq // G].T @ Wo[hq * d:(hq + 1) * d, :]
        # the three projections as one GEMM: [W_Q | W_K | W_V_hat], [hidden][(n_q + 2 n_kv) 128]
        self.W_qkv = torch.cat([W_q, W_k, Wv.to(self.dtype)], dim=1).contiguous()
        self.W_o_hat = Wo.to(self.dtype).contiguous()
        self.cache = swan.SwanCache(batch, n_heads, n_kv_heads, buffer_tokens, capacity,
                                    k_active, self.dtype, W_q.device,
                                    sparse_values=sparse_values, k_value=k_value)

    def project(self, x):
        """Post-RoPE q [B][H_q][n][128], k and v_hat [B][H_kv][n][128] of new rows x
        [B][n][hidden] at each sequence's next positions."""
        qkv = x @ self.W_qkv
        nq, nkv = self.n_heads * HEAD_DIM, self.n_kv_heads * HEAD_DIM
        return (self._rows(qkv[..., :nq], self.n_heads, True),
                self._rows(qkv[..., nq:nq + nkv], self.n_kv_heads, True),
                self._rows(qkv[..., nq + nkv:], self.n_kv_heads, False))

    def _rows(self, t, heads: int, rope: bool):
        """[B][n][heads 128] projections as [B][heads][n][128], rotated by RoPE at the
        sequences' next positions."""
        B, n, _ = t.shape
        t = t.reshape(B, n, heads, HEAD_DIM).transpose(1, 2).contiguous()
        if rope:
            swan.rope(t, self.cache.seq_len, self.rope_base, out=t)
        return t

    def _prompt_rows(self, x):
        """project(x) without the queries: a prompt's attention is not part of this layer,
        and for 32 query and 8 KV heads its keys and values are a third of the projections.
        Any other project() than this class's own is called as it is."""
        if getattr(self.project, "__func__", None) is not _OWN_PROJECT:
            return self.project(x)[1:]
        nq, nkv = self.n_heads * HEAD_DIM, self.n_kv_heads * HEAD_DIM
        kv = x @ self.W_qkv[:, nq:]
        return (self._rows(kv[..., :nkv], self.n_kv_heads, True),
                self._rows(kv[..., nkv:], self.n_kv_heads, False))

    def __call__(self, x):
        """x [B][n][hidden]: append the n rows of every sequence to the cache; for a
        decode step (n = 1) return y [B][hidden], the layer's attention output."""
        if x.shape[1] != 1:
            k, v = self._prompt_rows(x)
            self.cache.append(k, v, self.P_qk, None)
            return None
        q, k, v = self.project(x)
        B = x.shape[0]
        o_hat = self.cache.step(k, v, q[:, :, 0].contiguous(), self.P_qk, None)
        return o_hat.view(B, self.n_heads * HEAD_DIM) @ self.W_o_hat


_OWN_PROJECT = SwanAttentionLayer.project  # also when the class's is replaced
