"""PyTorch plumbing around the C ABI: device buffers and the current stream.

Nothing here computes: tensors are allocated with torch, raw pointers and the
stream handle go to the library, and every step of the path runs in its kernels.
"""
from __future__ import annotations

import numpy as np
import torch

from . import binding as B


# the raw handle of torch's current stream, without building a Stream object for it (3 us a launch) where torch offers that
_raw_stream = getattr(torch._C, "_cuda_getCurrentRawStream", None)


def _stream() -> int:
    if _raw_stream is not None:
        return _raw_stream(torch.cuda.current_device())
    return int(torch.cuda.current_stream().cuda_stream)


def to_device(bits: np.ndarray, dtype: str, device="cuda:0") -> torch.Tensor:
    """Stored bits (float32 / uint16 bf16 patterns / uint8 e4m3 codes) -> device tensor, bit for bit."""
    if dtype == "f32":
        return torch.from_numpy(np.ascontiguousarray(bits, np.float32)).to(device)
    if dtype == "bf16":
        return torch.from_numpy(np.ascontiguousarray(bits, np.uint16).view(np.int16)).to(device).view(torch.bfloat16)
    if dtype == "fp8_e4m3":
        return torch.from_numpy(np.ascontiguousarray(bits, np.uint8)).to(device)
    raise ValueError(dtype)


def from_device(t: torch.Tensor) -> np.ndarray:
    """Device tensor -> float64 numpy (bf16 widened exactly)."""
    return t.detach().to("cpu").to(torch.float64).numpy()


class DecodeBatch:
    """Device-side state of one decode batch: uploaded tables, workspace, Q, output."""

    def __init__(self, layout, geometry: B.ps_geometry, num_requests: int, q: torch.Tensor, kv: torch.Tensor,
                 scales: torch.Tensor | None = None):
        if not torch.cuda.is_available():
            raise RuntimeError("a GPU is required: the attention path has no CPU fallback")
        self.layout, self.geometry, self.num_requests = layout, geometry, num_requests
        self.q, self.kv, self.scales = q, kv, scales
        self.device = q.device
        self.out = torch.empty_like(q)
        self.lse = torch.empty((num_requests, geometry.num_q_heads), dtype=torch.float32, device=self.device)
        self.tables = None
        self.workspace = None
        self._sync_plan()

    def _sync_plan(self, wait=True, tokens=None):
        # (the layout has changed: where the new tables cannot be had, the old ones must not be launched from)
        old, self.tables, self.workspace = (self.tables, self.workspace), None, None
        self._home = _stream()               # tables and workspace belong to this stream
        tables = torch.empty(B.ps_layout_device_bytes(self.layout), dtype=torch.uint8, device=self.device)
        workspace = torch.empty(B.ps_workspace_bytes(self.layout), dtype=torch.uint8, device=self.device)
        del old
        self._pending = not wait             # other streams have to wait for the upload on the GPU
        if tokens is None:
            B.ps_layout_upload(self.layout, tables.data_ptr(), _stream())
        else:
            B.ps_layout_upload_append(self.layout, tables.data_ptr(), tokens[0].data_ptr(), tokens[1].data_ptr(),
                                      self.kv.data_ptr(), self._sc(), _stream())
        self.tables, self.workspace = tables, workspace
        if wait:
            torch.cuda.current_stream().synchronize()

    def replan(self, options: B.ps_plan_options | None):
        B.ps_layout_replan(self.layout, options)
        self._sync_plan()

    def set_visible(self, prefix_visible=None):
        """Limit how much of its prompt's shared prefix every request sees (None = all of it)."""
        B.ps_layout_set_visible(self.layout, self.num_requests, prefix_visible)
        self._sync_plan()

    def _stream(self) -> int:
        """The current stream, for a launch that reads the tables: behind their upload, whichever stream that went to, and
        they and the workspace live until the launch is done."""
        stream = _stream()
        if stream != self._home:
            current = torch.cuda.current_stream()
            # (a launch that is only recorded runs with the graph, whose replays the caller orders)
            if self._pending and not torch.cuda.is_current_stream_capturing():
                B.ps_layout_upload_wait(self.layout, stream)
            for t in (self.tables, self.workspace):
                t.record_stream(current)
        return stream

    def _sc(self):
        return self.scales.data_ptr() if self.scales is not None else 0

    def prefix_attention(self):
        B.ps_prefix_attention(self.layout, self.tables.data_ptr(), self.q.data_ptr(), self.kv.data_ptr(), self._sc(),
                              self.workspace.data_ptr(), self._stream())

    def suffix_attention(self):
        B.ps_suffix_attention(self.layout, self.tables.data_ptr(), self.q.data_ptr(), self.kv.data_ptr(), self._sc(),
                              self.workspace.data_ptr(), self._stream())

    def merge_states(self, with_lse=True):
        B.ps_merge_states(self.layout, self.tables.data_ptr(), self.workspace.data_ptr(), self.out.data_ptr(),
                          self.lse.data_ptr() if with_lse else 0, self._stream())

    def decode_attention(self, with_lse=True, kv: torch.Tensor | None = None):
        B.ps_decode_attention(self.layout, self.tables.data_ptr(), self.q.data_ptr(),
                              (self.kv if kv is None else kv).data_ptr(), self._sc(), self.workspace.data_ptr(),
                              self.out.data_ptr(), self.lse.data_ptr() if with_lse else 0, self._stream())

    def kv_ingest(self, which: int, src_k: torch.Tensor, src_v: torch.Tensor):
        """Store every segment of one kind (0 prefixes, 1 suffixes) from ragged [T, Hkv, d] sources."""
        assert src_k.stride(2) == 1 and src_v.stride() == src_k.stride()
        B.ps_kv_ingest(self.layout, self.tables.data_ptr(), which, src_k.data_ptr(), src_v.data_ptr(),
                       src_k.stride(0), src_k.stride(1), self.kv.data_ptr(), self._sc(), self._stream())

    def append_step(self, pool, new_k: torch.Tensor, new_v: torch.Tensor, active=None):
        """One decode step of cache growth: tables grow on the host and are uploaded again, then the new
        tokens ([R, Hkv, d], contiguous) are stored.  Returns the destinations the host chose."""
        if torch.cuda.is_current_stream_capturing():
            raise RuntimeError("append_step changes the tables on the host: it cannot be recorded into a graph")
        if not (new_k.is_contiguous() and new_v.is_contiguous()):
            raise ValueError("append_step stores tokens from contiguous tensors")
        dest = B.ps_layout_append(pool, self.layout, self.num_requests, active)
        # No wait on the host for the upload: it is ordered in front of what follows on this stream, and launches of this
        # batch on other streams wait for it there.
        self._sync_plan(wait=False, tokens=(new_k, new_v))
        return dest

    def stage_out(self, image: torch.Tensor):
        """Copy the batch's blocks (and e4m3 scales) into `image`: uint8, device memory or pinned host memory."""
        B.ps_kv_stage_out(self.layout, self.tables.data_ptr(), self.kv.data_ptr(), self._sc(), image.data_ptr(), self._stream())

    def stage_in(self, image: torch.Tensor):
        B.ps_kv_stage_in(self.layout, self.tables.data_ptr(), image.data_ptr(), self.kv.data_ptr(), self._sc(), self._stream())

    def park(self, pool):
        """Hand the batch's blocks back to the pool (after stage_out has completed)."""
        torch.cuda.current_stream().synchronize()
        B.ps_layout_park(pool, self.layout)

    def resume(self, pool):
        """Take blocks again and upload the new tables; stage_in then restores the contents."""
        B.ps_layout_resume(pool, self.layout)
        self._sync_plan()

    def workspace_views(self):
        """(o [slots, Hq, d] fp32, lse [slots, Hq] fp32) views of the partial-state workspace."""
        slots, off = B.ps_workspace_layout(self.layout)
        g = self.geometry
        o = self.workspace[:off].view(torch.float32).view(slots, g.num_q_heads, g.head_dim)
        lse = self.workspace[off:off + slots * g.num_q_heads * 4].view(torch.float32).view(slots, g.num_q_heads)
        return o, lse
