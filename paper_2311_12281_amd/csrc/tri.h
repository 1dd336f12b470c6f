// Internal: the triangle path, which computes the closed counts of all edges
// at once from the triangles of the graph (tri.hip) instead of intersecting
// the neighbour lists of one edge after another.
#pragma once

#include "scan_internal.h"

namespace scan {

// Vertices are renamed by decreasing degree (ties by id): h = 0 is the vertex
// of the highest degree.  In a batch (a disjoint union) every graph keeps its
// range of ids and is renamed inside it, so that its rows stay together.  Every edge is kept once, in the row of its endpoint
// with the larger h: row u lists the neighbours v of u with h(v) < h(u), in
// decreasing order.  No row is longer than about sqrt(2 m).
//
// Rows are cut into lines of 32 entries, aligned to lines; an entry holds h + 1
// of its neighbour, 0 where the last line has none.
// An entry is addressed by its place 32 * line + column everywhere: its
// neighbour (oc), its count (cnt), and one bit of simw[line].
constexpr int kTriLine = 32;
constexpr int kTriMaxRow = 4096;  // longest row the kernels take
constexpr int kTriBlock = 512;    // threads of the block kernel
constexpr int kTriRecLines = 8;   // lines per in-edge record
constexpr int kTriBatch = 56;     // records a wave decodes together; up to 7 more are asked for, and are empty
constexpr int kTriJob = 2 * kTriBatch * (kTriBlock / 64);  // records per job of the block kernel
constexpr int kTriDirect = 16384; // h below this: table of row positions indexed by h
constexpr int kTriShort = 65534;  // h below this: 16-bit entries (oc16) and a bitmap table
constexpr int kTriWaveRow = 128;  // rows up to this, with few in-edges, go one per wave
constexpr int kTriWaveSlots = 256;
constexpr uint32_t kTriWaveSingle = 1u << 31;  // the wave has all of them: counts are stored, not added
constexpr int64_t kTriWaveWords = 512;  // words of in-edges a wave takes on

// A line as the close kernel reads it.
struct TriLineInfo {
  int32_t u;        // the row's vertex
  uint32_t wbase;   // first bit word of the row
  int32_t deg;      // degree of u
  uint32_t shape;   // row length | column of the line << 16
};

// Lines of one in-edge (u, v) of a vertex v, up to kTriRecLines for the block
// kernel, one for the wave kernel: the columns of
// row u after v's entry are the w to look up in row v.
struct TriRec {
  uint32_t line;  // first line (of v's entry in row u, or a later one)
  uint32_t word;  // bit word of that line
  uint32_t nw;    // lines
  int32_t v;      // the vertex (read by k_tri_few only)
};

struct TriJob {
  int32_t v;
  uint32_t rbeg, rcnt;  // in-edge records
  uint32_t single;      // 1: the only job of v (its counts are stored, not added)
};

// A vertex of the wave kernel, or a part of its records (of one line each).
struct TriWave {
  int32_t v;
  uint32_t line, rbeg;  // of its row, of its in-edge records
  uint32_t shape;       // row length | records << 8 | kTriWaveSingle
};

// The graphs of a batch: vertices vtx_off[k] .. vtx_off[k + 1] - 1, and the
// graph of every vertex (the same array by id and by h).  All null for one graph.
struct TriGroups {
  int32_t count = 0;
  const int64_t* h_vtx_off = nullptr;  // host
  const int64_t* vtx_off = nullptr;    // device
  const int32_t* gid = nullptr;        // device
};

// Read-only after creation.
struct TriLayout {
  int32_t n = 0;
  int32_t span = 0;           // vertices of the largest graph
  const int64_t* vtx_off = nullptr;  // TriGroups (not owned)
  const int32_t* gid = nullptr;
  int64_t lines = 0, words = 0, recs = 0, steps = 0;
  int64_t jobs = 0, wave_rows = 0;
  int64_t few_at = 0, few = 0;  // records of the vertices of at most kNarrowRow neighbours, unused ones among them
  int32_t max_row = 0, max_hash_row = 0;
  int32_t* hof = nullptr;     // [n] id -> h
  int32_t* idof = nullptr;    // [n] h -> id
  int32_t* deg = nullptr;     // [n] degree, by h
  int32_t* row = nullptr;     // [n] entries of a row, by h
  uint32_t* oline = nullptr;  // [n + 1] first line of a row
  uint32_t* wbase = nullptr;  // [n + 1] first bit word of a row
  int32_t* lu = nullptr;      // [lines] h of the line's row
  TriLineInfo* li = nullptr;  // [lines]
  int32_t* oc = nullptr;      // [32 lines + pad] h + 1 of the neighbour, or 0
  uint16_t* oc16 = nullptr;   // the same within the graph in 16 bits, 0xFFFF for h >= kTriShort
  TriRec* rec = nullptr;      // [recs] a vertex's records, then unused ones
  TriJob* job = nullptr;      // [jobs], hubs first
  void* mem[4] = {};  // per vertex; rows; rows' 16-bit form and records; jobs
  TriWave* wrow = nullptr;    // [wave_rows]
};

// Written by every run.
struct TriScratch {
  int32_t* cnt = nullptr;     // [32 lines] common neighbours, then closed counts
  uint32_t* bits = nullptr;   // [words]
  uint32_t* simw = nullptr;   // [lines] similar entries
  int32_t* flag = nullptr;    // [1] some vertex is a core
  void* mem = nullptr;        // holds bits, simw and flag
};

// Device bytes held by the layout and by one scratch.
uint64_t tri_layout_bytes(const TriLayout& T);
uint64_t tri_scratch_bytes(const TriLayout& T, const TriScratch& S);

// Builds the layout from a validated CSR on the device (h_rp: the caller's
// offsets; csr: what check_csr found).  *ok = 0 with hipSuccess when the graph is outside the path's
// limits, or the layout and `scratches` scratches would take more than max_bytes
// (nothing stays allocated).  bucket_edges: edges per degree bucket.
hipError_t tri_build(hipStream_t s, int32_t n, int64_t nnz, const int64_t* h_rp, const int64_t* d_rp,
                     const int32_t* d_ci, const LayoutResult& csr, const TriGroups* groups, int scratches,
                     uint64_t max_bytes, TriLayout* T, int64_t* bucket_edges, int* ok);
void tri_release(TriLayout& T);
hipError_t tri_alloc_scratch(const TriLayout& T, TriScratch* S);
// Lays a scratch out at base (256-byte aligned; S null: to size only), which stays
// the caller's; its bytes.
uint64_t tri_place_scratch(const TriLayout& T, unsigned char* base, TriScratch* S);
void tri_release_scratch(TriScratch& S);
void tri_drop_work(TriScratch& S);  // all but the counts

// eps = p/q and mu of a run, or of every graph of a batch (q == 0 and no gq:
// only the closed counts, left in S.cnt).
struct TriArgs {
  uint64_t p = 0, q = 0;
  int32_t mu = 2;
  const int32_t* gid = nullptr;  // null: one graph
  const uint64_t* gp = nullptr;
  const uint64_t* gq = nullptr;
  const int32_t* gmu = nullptr;
};

// Kernel launches of the phases, in this order.  With the counts at hand, a
// query starts with tri_init_state and tri_threshold instead of the first three.
void tri_init_state(hipStream_t s, const TriLayout& T, const TriScratch& S, int32_t* lower, int32_t* parent,
                    int32_t* label, uint8_t* role);
void tri_threshold(hipStream_t s, const TriLayout& T, const TriScratch& S, const TriArgs& a, int32_t* lower);
// Frees what only the counting reads.
void tri_drop_inputs(TriLayout& T);
void tri_init(hipStream_t s, const TriLayout& T, const TriScratch& S, int32_t* lower, int32_t* parent,
              int32_t* label, uint8_t* role);
void tri_count(hipStream_t s, const TriLayout& T, const TriScratch& S);
void tri_close(hipStream_t s, const TriLayout& T, const TriScratch& S, const TriArgs& a, int32_t* lower);
void tri_hook(hipStream_t s, const TriLayout& T, const TriScratch& S, const TriArgs& a, const int32_t* lower,
              int32_t* parent);
void tri_attach(hipStream_t s, const TriLayout& T, const TriScratch& S, const TriArgs& a, const int32_t* lower,
                int32_t* parent, int32_t* label);
// Hub marks (Def 2.7): role[id] = ROLE_HUB; first is scratch of n entries.
void tri_hub_outlier(hipStream_t s, const TriLayout& T, const TriScratch& S, const TriArgs& a, const int32_t* lower,
                     int32_t* parent, int32_t* label, int32_t* first, uint8_t* role);
void tri_output(hipStream_t s, const TriLayout& T, const TriArgs& a, const int32_t* lower, int32_t* parent,
                const int32_t* label, const uint8_t* role, int32_t* out_labels, uint8_t* out_roles, int32_t split);
// Closed counts of every arc in CSR order from S.cnt (after tri_close).
void tri_arc_counts(hipStream_t s, const TriLayout& T, const TriScratch& S, int64_t nnz, const int64_t* rp,
                    const int32_t* ci, int32_t* counts);

}  // namespace scan
