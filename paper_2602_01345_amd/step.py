"""One next-scale step through L entropy-pruned blocks: a sequence of C-ABI calls.

For every block j:  nova_entropy -> nova_select -> nova_pruned_block -> nova_merge_cache,
all enqueued on the current stream with no host synchronisation in between (the keep
count k_j is an input).  The entropies and selections read the blocks' logits only, inputs of the step like the
keep counts, so a step takes them for all blocks first, up to 32 per launch (nova_entropy_blocks, nova_select_blocks).
This module only owns device buffers and call order.
"""
from __future__ import annotations

from dataclasses import dataclass, field
from typing import Dict, List, Optional

import torch

from .binding import NOVA_BF16, NOVA_F32, BlockShape, BlockVariant, Nova


@dataclass
class BlockState:
    """Device-resident inputs and outputs of one block at one step."""
    k: int
    logits: torch.Tensor                 # [B, N, V]
    weights: Dict[str, torch.Tensor]
    k_cache: torch.Tensor                # [B, heads, cap, dh]
    v_cache: torch.Tensor                # [B, heads, dh, cap]
    cache_prev: Optional[torch.Tensor]   # [B, hp*wp, C]
    entropy: torch.Tensor = None         # [B, N] f32
    kept_idx: torch.Tensor = None        # [B, k] i32
    keep_mask: torch.Tensor = None       # [B, N] u8
    y_kept: torch.Tensor = None          # [B, k, C]
    out: torch.Tensor = None             # [B, N, C]
    cache_new: torch.Tensor = None       # [B, N, C]
    variant: Optional[BlockVariant] = None   # block variations (nova_pruned_block_variant); None = the base block


class StepRunner:
    def __init__(self, nova: Nova, *, B: int, grid: int, prev_grid: int, C: int, heads: int, kv_len: int,
                 kv_capacity: int, dtype: torch.dtype, ffn_mult: int = 4):
        self.nova = nova
        self.B, self.grid, self.prev_grid, self.C, self.heads = B, grid, prev_grid, C, heads
        self.N = grid * grid
        self.kv_len, self.kv_capacity, self.ffn_mult = kv_len, kv_capacity, ffn_mult
        self.dtype = dtype
        self.code = NOVA_BF16 if dtype == torch.bfloat16 else NOVA_F32
        self.blocks: List[BlockState] = []
        self._workspace: Optional[torch.Tensor] = None
        self._side: Optional[torch.cuda.Stream] = None      # second stream for the look-ahead selection
        self._selected: List[torch.cuda.Event] = []
        self._started: List[torch.cuda.Event] = []

    def shape(self, k: int) -> BlockShape:
        return BlockShape(self.code, self.B, self.N, self.C, self.heads, self.kv_len, self.kv_capacity, k,
                          self.ffn_mult)

    def add_block(self, st: BlockState) -> BlockState:
        dev = st.logits.device
        B, N, C = self.B, self.N, self.C
        st.entropy = torch.empty((B, N), dtype=torch.float32, device=dev)
        st.kept_idx = torch.empty((B, max(st.k, 1)), dtype=torch.int32, device=dev)
        st.keep_mask = torch.empty((B, N), dtype=torch.uint8, device=dev)
        st.y_kept = torch.empty((B, max(st.k, 1), C), dtype=self.dtype, device=dev)
        st.out = torch.empty((B, N, C), dtype=self.dtype, device=dev)
        st.cache_new = torch.empty((B, N, C), dtype=self.dtype, device=dev)
        need = self.nova.workspace_bytes(self.shape(st.k))
        if self._workspace is None or self._workspace.numel() < need:
            self._workspace = torch.empty(max(need, 256), dtype=torch.uint8, device=dev)
        self.blocks.append(st)
        return st

    def run_block(self, st: BlockState, x: torch.Tensor) -> torch.Tensor:
        n = self.nova
        n.entropy(st.logits, st.entropy)
        n.select(st.entropy, st.k, st.kept_idx, st.keep_mask)
        if st.variant is None:
            n.pruned_block(self.shape(st.k), st.weights, x, st.kept_idx, st.k_cache, st.v_cache, st.y_kept,
                           self._workspace)
        else:
            n.pruned_block_variant(self.shape(st.k), st.weights, st.variant, x, st.kept_idx, st.k_cache,
                                   st.v_cache, st.y_kept, self._workspace)
        n.merge_cache(self.grid, self.grid, self.prev_grid, self.prev_grid, st.k, x, st.y_kept, st.kept_idx,
                      st.keep_mask, st.cache_prev, st.out, st.cache_new)
        return st.out

    def _select(self, st: BlockState) -> None:
        self.nova.entropy(st.logits, st.entropy)
        self.nova.select(st.entropy, st.k, st.kept_idx, st.keep_mask)

    def _block_and_merge(self, st: BlockState, x: torch.Tensor) -> torch.Tensor:
        n = self.nova
        if st.variant is None:
            n.pruned_block(self.shape(st.k), st.weights, x, st.kept_idx, st.k_cache, st.v_cache, st.y_kept,
                           self._workspace)
        else:
            n.pruned_block_variant(self.shape(st.k), st.weights, st.variant, x, st.kept_idx, st.k_cache,
                                   st.v_cache, st.y_kept, self._workspace)
        n.merge_cache(self.grid, self.grid, self.prev_grid, self.prev_grid, st.k, x, st.y_kept, st.kept_idx,
                      st.keep_mask, st.cache_prev, st.out, st.cache_new)
        return st.out

    def run_step(self, x: torch.Tensor, overlap_selection: bool = False) -> torch.Tensor:
        """All blocks of the step: entropies and selections of all of them, then block after block.  With
        overlap_selection each block's entropy and selection, which read that block's logits only, are launches of
        their own instead, enqueued one block ahead on a second stream (default priority) next to the previous
        block's gather and QKV projection.  The values are the same either way.  Off by default: on the largest
        workload a step takes 20.7 ms with it and 20.3 without (the launches of single blocks are mostly ramp and
        tail, and the entropy kernel fills the CUs, so the two streams mostly take turns)."""
        if len(self.blocks) < 2:
            for st in self.blocks:
                x = self.run_block(st, x)
            return x
        if not overlap_selection:
            bs = self.blocks
            self.nova.entropy_blocks([st.logits for st in bs], [st.entropy for st in bs])
            self.nova.select_blocks([st.entropy for st in bs], [st.k for st in bs], [st.kept_idx for st in bs],
                                    [st.keep_mask for st in bs])
            for st in bs:
                x = self._block_and_merge(st, x)
            return x
        main = torch.cuda.current_stream()
        if self._side is None:
            self._side = torch.cuda.Stream()
        while len(self._selected) < len(self.blocks):
            self._selected.append(torch.cuda.Event())
            self._started.append(torch.cuda.Event())
        side = self._side
        self._select(self.blocks[0])
        for j, st in enumerate(self.blocks):
            if j + 1 < len(self.blocks):
                # the look-ahead starts when block j starts (not earlier: the host runs far ahead of the device),
                # so it lands next to block j's gather and QKV projection
                self._started[j].record(main)
                with torch.cuda.stream(side):
                    side.wait_event(self._started[j])
                    self._select(self.blocks[j + 1])
                    self._selected[j + 1].record(side)
            if j > 0:
                main.wait_event(self._selected[j])
            x = self._block_and_merge(st, x)
        return x
